// Per-document count (one table per document; the paper's per-document dictionaries of
// Section 3.1, before the grouping of Section 3.3).
//
// Work. The corpus is cut into windows; a window owns the documents whose first byte lies in it. A
// document longer than the window is always its last one; such documents are counted alone, the
// rest of a window up to kDocW documents at a time ("group"). doc_plan_kernel lists the groups by
// size class; persistent workgroups (1024 threads, one per CU) take them from a queue, the
// largest class first.
//
// Counting. A group's text is cut into tiles of 992 bytes, staged with the 16 bytes before and after;
// a wave that has counted one takes the next that is left (no workgroup barrier inside the scan; with
// equal runs of whole stripes for the waves 19 % of the time went by with the last of them alone).
// A token's document is its index r in the group, found from the tile's document starts; (word, r) is one 16-byte key in the
// LDS table of wc_words.h: r sits in bit 7 of the bytes of a packed word's second half, bits that
// no word byte uses, or above the 48 address bits of a long word. Most groups fit the table. A
// token whose key finds no entry left is spilled: its key goes to a chunk of records in device
// memory (each wave fills its own chain of chunks). After the scan, spilled keys that do have an
// entry (a lane can be refused while another wave publishes the same word) are counted in it, the
// table's entries are set aside in device memory, the table is emptied, and the rest is counted
// in it: at once if it must fit, and otherwise split by hash into 256 parts, as many parts to a
// table as must fit. A part that does not fit by itself spills again. So a key is in one table
// only, and a document of any size costs a fixed number of passes over what its words spilled.
//
// Device memory for that is taken in regions, which a workgroup keeps for its later groups: 16 of
// 1,024 slots, 16 of 2,048, and so on, so that no more than a sixteenth goes unused. They are
// addressed as one space ("virtual" slots) that starts anew with each group.
//
// Output. Every entry takes its (entry, byte) place inside its document with one 64-bit LDS atomic;
// one 64-bit atomic add on a packed cursor (entries << 32 | bytes) reserves space for the group;
// then the entries in LDS, and those set aside, are written, so every document's entries and word
// bytes are contiguous and the word offsets stay a valid CSR over the whole output.
//
// What a group waits for is taken early: the queue position after the next group's is asked for by
// the first wave that ends its scan, its offsets are read while this group's entries find their
// places, and the next group's first text is loaded before this group's entries are written.
//
// Bound by instructions: vector units are busy for 65 % of the time; a third of it is the table (and
// what spills), a fifth taking the words apart, a tenth writing the output, a sixth finding words,
// and the rest the waits inside a group and between them. Two
// workgroups per CU with half the table each were slower (more and smaller groups, more spills).
// 100,000 documents (lognormal, median 16 KiB, 2.7 GB, 119 million entries), before as two passes
// with tables of 4,096 entries in LDS and in device memory: 12.7 -> 5.5 ms; 2,000 documents of 2 to
// 20 KiB: 181 -> 74 us.
//
// Every size the kernels need is read from a device-side task description, so a whole call
// can be captured once in a HIP graph and replayed for other corpora.
#include <type_traits>

#include "wc_internal.h"
#include "wc_stripe.h"
#include "wc_words.h"

namespace wc {

namespace {

constexpr int kBlk = 1024;
constexpr uint32_t kWaves = kBlk / 64;
constexpr uint32_t kTile = kStripe - 32;      // bytes whose words a wave counts at a time
constexpr uint32_t kText = kStripe + 32;      // per wave: a tile with 16 bytes on each side, padding
constexpr uint32_t kList = 192;               // starts of a tile listed at a time (256: 100 table
                                              // entries fewer, 100,000 documents 5.44 ms for 5.37)
constexpr uint32_t kEnds = kStripe / 32 + 2;  // word-end bitmap of the staged text, two words of zeros
constexpr uint32_t kListWords = kList / 2 + kEnds;
constexpr uint32_t kPerThread = (kDocLds + kBlk - 1) / kBlk;
// spilled keys: a chunk is a link to the wave's chunk before it and kChunkRecs keys
constexpr uint32_t kChunkSlots = 128;
constexpr uint32_t kChunkRecs = kChunkSlots * sizeof(Slot) / 16 - 1;
constexpr uint32_t kDocParts = 256;
// regions of device memory: 16 of kUnit slots, 16 of twice as many, ...
constexpr uint32_t kUnit = 1024, kClassesMax = 20;
constexpr uint32_t kTaking = 0xfffffffeu, kNoRegion = 0xffffffffu;

// A work item: documents << kItemShift | the first one.
constexpr uint32_t kItemShift = 48;
WC_DEV uint32_t item_docs(uint64_t it) { return (uint32_t)(it >> kItemShift); }
WC_DEV uint64_t item_first(uint64_t it) { return it & ((1ull << kItemShift) - 1); }

// bits 0..3 of n -> bits 7, 15, 23, 31 (the top bits of four bytes)
WC_DEV uint32_t spread4(uint32_t n) {
  return (__umul24(n & 7u, 0x204080u) & 0x808080u) | ((n & 8u) << 28);
}
// bits 7, 15, 23, 31 -> bits 0..3
WC_DEV uint32_t gather4(uint32_t x) {
  return ((x >> 7) & 1u) | ((x >> 14) & 2u) | ((x >> 21) & 4u) | ((x >> 28) & 8u);
}
// A key of document r (< 256), its document, and the word's key without it.
WC_DEV uint4 with_doc(uint4 k, uint32_t r) {
  if (is_long_key(k)) {
    k.y |= r << 16;
  } else {
    k.z |= spread4(r & 15u);
    k.w |= spread4(r >> 4);
  }
  return k;
}
WC_DEV uint32_t key_doc(const uint4 k) {
  return is_long_key(k) ? k.y >> 16 : gather4(k.z) | (gather4(k.w) << 4);
}
WC_DEV uint4 without_doc(uint4 k) {
  if (is_long_key(k)) {
    k.y &= 0xffffu;
  } else {
    k.z &= 0x7f7f7f7fu;
    k.w &= 0x7f7f7f7fu;
  }
  return k;
}

}  // namespace

constexpr size_t kDyn = (size_t)kDocSlots * 4 + (size_t)kDocLds * 20 + (size_t)kWaves * kText;

// (the parameters are read with args(): as an argument by name they would be loaded once, at the
// start, and held or spilled over the scan: 50 of its instructions per KiB read such values back)
__global__ __launch_bounds__(kBlk) void doc_kernel(DocParams) {
  typedef const __attribute__((address_space(4))) DocParams* Args;
  auto args = []() -> Args {
    Args a = (Args)__builtin_amdgcn_kernarg_segment_ptr();
    __asm__ volatile("" : "+s"(a));
    return a;
  };

  extern __shared__ __align__(16) uint8_t s_dyn[];
  __shared__ uint32_t s_list[kWaves][kListWords];  // starts (16 bits each), then the end bitmap
  __shared__ uint32_t s_bnd[kWaves][kEnds];        // document starts of a tile
  __shared__ uint4 s_lenmask[17];
  __shared__ uint64_t s_doff[3][kDocW + 1];        // document offsets of the group and the next two
  __shared__ unsigned long long s_dcur[kDocW];     // places taken: (entries << 32 | bytes)
  __shared__ uint32_t s_sum[4], s_class[kDocClasses + 1];
  __shared__ uint64_t s_out;
  __shared__ unsigned long long s_tokens;
  __shared__ uint32_t s_nent, s_spill, s_next, s_done, s_tile;
  __shared__ uint32_t s_region[16 * kClassesMax];  // first unit + 1 (0: not taken yet)
  __shared__ uint32_t s_part[kDocParts];
  __shared__ uint32_t s_used, s_lost, s_at;         // virtual slots used; some region was refused

  const uint32_t tid = threadIdx.x, lane = tid & 63;
  const uint32_t wv = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
  auto hdr_of = [&]() -> Header* { return as_global(args()->hdr); };

  const uint8_t* const corpus = as_global(as_global(args()->task)->corpus);
  const uint64_t len = uniform64(as_global(args()->task)->len);
  auto offset_at = [&](uint64_t d) -> uint64_t { return as_global(as_global(args()->task)->offsets)[d]; };
  const int64_t base_off = -(int64_t)((uintptr_t)corpus & 15);
  if (ld_relaxed32(&hdr_of()->flags) & kFlagBadOffsets) return;

  PartTable<uint32_t, kDocSlots> T;
  T.slot = (uint32_t*)s_dyn;
  T.key = (uint4*)(T.slot + kDocSlots);
  T.cnt = (uint32_t*)(T.key + kDocLds);
  T.n = &s_nent;
  T.cap = (uint32_t)uniform64(min(args()->lds_cap, kDocLds));
  uint8_t* const my_txt = (uint8_t*)(T.cnt + kDocLds) + wv * kText;
  uint16_t* const my_starts = (uint16_t*)s_list[wv];
  uint32_t* const my_ends = s_list[wv] + kList / 2;
  uint32_t* const my_bnd = s_bnd[wv];

  for (uint32_t i = tid; i < kWaves * kListWords; i += kBlk) (&s_list[0][0])[i] = 0;
  for (uint32_t i = tid; i < kWaves * kEnds; i += kBlk) (&s_bnd[0][0])[i] = 0;
  for (uint32_t i = tid; i < 16 * kClassesMax; i += kBlk) s_region[i] = 0;
  if (tid == 0) s_lost = 0;
  init_len_masks(s_lenmask, tid, kBlk);
  for (uint32_t r = tid; r < kDocW; r += kBlk) s_dcur[r] = 0;
  auto clear_slots = [&]() {
    for (uint32_t i = tid; i < kDocSlots / 4; i += kBlk) ((uint4*)T.slot)[i] = make_uint4(0, 0, 0, 0);
  };
  clear_slots();

  // ---- device memory of the group ----------------------------------------------------------
  auto region_of = [&](uint32_t v, uint32_t* start) -> uint32_t {
    const uint32_t u = v / kUnit, c = 31u - (uint32_t)__clz((int)(u / 16 + 1));
    const uint32_t w = (u - 16 * ((1u << c) - 1)) >> c;
    *start = (16 * ((1u << c) - 1) + (w << c)) * kUnit;
    return c * 16 + w;
  };
  auto slot_at = [&](uint32_t v) -> Slot* {
    uint32_t start;
    const uint32_t i = region_of(v, &start);
    return as_global(args()->arena) + (uint64_t)(s_region[i] - 1) * kUnit + (v - start);
  };
  // the region of virtual slot v is taken by one lane; the others wait for it. False: refused
  auto ensure = [&](uint32_t v) -> bool {
    uint32_t start;
    const uint32_t i = region_of(v, &start);
    uint32_t r = atomicCAS(&s_region[i], 0u, kTaking);
    if (r == 0) {
      const uint64_t size = (uint64_t)kUnit << (i / 16);
      const uint64_t at = atomicAdd((unsigned long long*)&hdr_of()->arena_next, (unsigned long long)size);
      r = at + size <= args()->arena_slots ? (uint32_t)(at / kUnit) + 1 : kNoRegion;
      atomicExch(&s_region[i], r);
    }
    while (r == kTaking) {
      __builtin_amdgcn_s_sleep(1);
      r = atomicOr(&s_region[i], 0u);
    }
    if (r == kNoRegion) {
      or32(&hdr_of()->flags, kFlagWordCap);
      atomicOr(&s_lost, 1u);
    }
    return r != kNoRegion;
  };
  // one thread's: n virtual slots
  auto take = [&](uint32_t n) -> uint32_t {
    const uint32_t v = s_used;
    n = (n + kChunkSlots - 1) & ~(kChunkSlots - 1);  // (a chunk lies in one region)
    s_used = v + n;
    for (uint32_t u = v / kUnit; u <= (v + n - 1) / kUnit; ++u) ensure(u * kUnit);
    return v;
  };

  // ---- spilled keys of this wave -----------------------------------------------------------
  uint32_t chunk = 0;    // the chain's last chunk: its virtual slot + 1 (0: none)
  uint32_t chunk_n = 0;  // keys in it (those before it are full)
  // the keys of NX tokens per lane, where left
  auto spill = [&](const uint4* key, const bool* left, auto nx) {
    constexpr int NX = decltype(nx)::value;
    uint32_t at[NX], total = 0;
#pragma unroll
    for (int x = 0; x < NX; ++x) {
      const uint64_t m = __ballot(left[x]);
      at[x] = total + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
      total += (uint32_t)__popcll(m);
    }
    for (uint32_t done = 0; done < total;) {
      if (!chunk || chunk_n == kChunkRecs) {
        uint32_t c = 0;
        if (lane == 0) {
          c = atomicAdd(&s_used, kChunkSlots);
          if (ensure(c)) *(uint4*)slot_at(c) = make_uint4(chunk, 0, 0, 0);
          s_spill = 1;
        }
        chunk = (uint32_t)__builtin_amdgcn_readfirstlane((int)c) + 1;
        chunk_n = 0;
      }
      const uint32_t n = min(kChunkRecs - chunk_n, total - done);
      if (!s_lost) {
        uint4* const rec = (uint4*)slot_at(chunk - 1) + 1 + chunk_n;
#pragma unroll
        for (int x = 0; x < NX; ++x)
          if (left[x] && at[x] - done < n) rec[at[x] - done] = key[x];
      }
      chunk_n += n;
      done += n;
    }
    wait_vmem();
  };

  // ---- the scan of documents [0, nd) of the group at doff ----------------------------------
  uint32_t tokens = 0;
  // The text [A, B) in tiles of kTile bytes, staged with the 16 bytes before and after them: a lane
  // reads 16 bytes, the first and the last lane for what the others' words touch. Tile k, from the
  // first 16-byte block on; bytes outside the text may be anything.
  auto tile_at = [&](int64_t A, uint32_t k) -> int64_t { return A - ((A - base_off) & 15) + (int64_t)k * kTile; };
  auto load = [&](int64_t A, int64_t B, uint32_t k) -> uint4 {
    const int64_t p = tile_at(A, k) - 16;
    uint4 v = make_uint4(0x20202020u, 0x20202020u, 0x20202020u, 0x20202020u);
    if (p + 16 >= B) return v;
    uint32_t at = lane * 16;
    pin(at);  // (an offset to a scalar address: as a sum of its own it was kept, and spilled)
    if (p >= 0 && p + (int64_t)kStripe <= (int64_t)len) v = load_stream16(corpus + p + at);
    else v = load_text16(corpus, len, p + at);
    return v;
  };
  uint4 t0 = make_uint4(0, 0, 0, 0);  // the wave's first tile of the next group, loaded a group ahead
  auto scan = [&](const uint64_t* doff, uint32_t nd) {
    const int64_t A = (int64_t)uniform64(doff[0]), B = (int64_t)uniform64(doff[nd]);
    // (the group's first 64 document starts in the lanes)
    const int64_t o0 = lane < nd ? (int64_t)doff[min(lane, nd)] : INT64_MAX;
    uint4 raw = t0;
    uint32_t spare[2] = {kNone, kNone};
    for (uint32_t k = wv; tile_at(A, k) < B;) {
      // the next tile is whichever no wave has taken
      uint32_t kn = 0;
      if (lane == 0) kn = atomicAdd(&s_tile, 1u);
      const int64_t pk = tile_at(A, k), p0 = pk - 16;
      uint32_t w16;
      const uint4 g = classify16(raw, &w16);
      if (p0 < A || p0 + (int64_t)kStripe > B) w16 = cut16(w16, p0 + lane * 16, A, B);
      ((uint4*)my_txt)[lane] = g;
      kn = (uint32_t)__builtin_amdgcn_readfirstlane((int)kn);
      raw = load(A, B, kn);
      // rb: the last document that starts before the tile (-1: none), nb: starts in it; a bit for
      // each start in it and the 16 bytes after it
      int32_t rb = -1;
      uint32_t bnd16 = 0, bnext = 0, nb = 0;
      bool some = false;
      for (uint32_t j = 0; j < nd; j += 64) {
        const int64_t o = j == 0 ? o0 : j + lane < nd ? (int64_t)doff[j + lane] : INT64_MAX;
        const uint64_t before = __ballot(o < pk), reach = __ballot(o < pk + kTile + 16);
        rb += (int32_t)__popcll(before);
        if (reach != before) {
          some = true;
          nb += (uint32_t)__popcll(__ballot(o < pk + kTile) & ~before);
          if (o >= pk && o < pk + kTile + 16)
            atomicOr(&my_bnd[(uint32_t)(o - p0) >> 5], 1u << ((uint32_t)(o - p0) & 31));
        }
        if (reach != ~0ull) break;
      }
      if (some) {
        wave_sync();
        bnd16 = (my_bnd[lane >> 1] >> ((lane & 1) * 16)) & 0xffffu;
        bnext = (my_bnd[(lane + 1) >> 1] >> (((lane + 1) & 1) * 16)) & 1u;  // lane 63: 0
        wave_sync();
        if (lane < kEnds) my_bnd[lane] = 0;
      }
      const uint32_t prev = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(w16 >> 15), 0x138, 0xf, 0xf, false);
      // (lane 63: a word that reaches the last byte started 16 bytes before it, and goes on for all
      // that is known: longer than 16 bytes)
      const uint32_t next = (uint32_t)__builtin_amdgcn_update_dpp(1, (int)(w16 & 1u), 0x130, 0xf, 0xf, false);
      uint32_t start16 = w16 & (~((w16 << 1) | prev) | bnd16) & 0xffffu;
      if (lane - 1 >= kTile / 16) start16 = 0;  // another tile's
      const uint32_t last16 = w16 & (~((w16 >> 1) | (next << 15)) | (bnd16 >> 1) | (bnext << 15)) & 0xffffu;
      ((uint16_t*)my_ends)[lane] = (uint16_t)last16;
      const uint32_t c = __popc(start16), incl = wave_incl_scan(c);
      const uint32_t n = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
      tokens += n;
      // document of the token at staged byte s: the last one that starts at or before it (empty
      // documents share their start with the next one); only the nb starts of the tile follow rb
      auto doc_at = [&](uint32_t s) -> uint32_t {
        int32_t a = rb, b = rb + 1 + (int32_t)nb;  // doff[a] <= p0 + s < doff[b]
        while (b - a > 1) {
          const int32_t m = (a + b) >> 1;
          if ((int64_t)doff[m] <= p0 + (int64_t)s) a = m;
          else b = m;
        }
        return a < 0 ? 0u : (uint32_t)a;
      };
      // key of a word longer than 16 bytes; wl: its length, or 0 when its end is not within 32 bytes
      auto long_word = [&](uint32_t s, uint32_t wl, uint32_t r) -> uint4 {
        const uint64_t start = (uint64_t)(p0 + s);
        for (uint32_t w = (s + 32) >> 5; !wl && w < kEnds; ++w) {
          uint32_t m = my_ends[w];
          if (w == (s + 32) >> 5) m &= 0xffffffffu << (s & 31);
          if (m) wl = w * 32 + __ffs(m) - s;
        }
        if (wl) {
          const uint32_t* tw = (const uint32_t*)my_txt;
          uint32_t h = wl;
          for (uint32_t q = 0; q < wl; q += 4) {
            const uint32_t at = s + q;
            uint32_t d = __builtin_amdgcn_alignbyte(tw[(at >> 2) + 1], tw[at >> 2], at & 3);
            if (wl - q < 4) d &= (1u << (8 * (wl - q))) - 1u;
            h = long_step(h, d);
          }
          return long_key(corpus + start, wl, h);
        }
        wl = (uint32_t)long_len(corpus, len, start, doff[r + 1]);
        return long_key(corpus + start, wl, long_hash(corpus + start, wl));
      };

      // the NX * 64 listed tokens from place `at` on; `nw` of them are there
      auto count = [&](auto nx, uint32_t at, uint32_t nw) {
        constexpr int NX = decltype(nx)::value;
        uint32_t st[NX], wl[NX], e0[NX], e1[NX], doc[NX], one[NX], h[NX];
        bool in[NX], left[NX];
        // (starts past nw are of earlier lists: in range, not counted)
#pragma unroll
        for (int x = 0; x < NX; ++x) st[x] = my_starts[at + lane + 64 * x];
#pragma unroll
        for (int x = 0; x < NX; ++x) {
          e0[x] = my_ends[st[x] >> 5];
          e1[x] = my_ends[(st[x] >> 5) + 1];
        }
#pragma unroll
        for (int x = 0; x < NX; ++x) {
          wl[x] = __ffs(__builtin_amdgcn_alignbit(e1[x], e0[x], st[x] & 31));  // 0: no end in 32
          in[x] = lane + 64 * x < nw;
          one[x] = 1;
        }
        // each LDS step reads for all tokens before any waits (pin)
        PackSrc ps[NX];
        uint4 lm[NX], key[NX];
#pragma unroll
        for (int x = 0; x < NX; ++x) {
          ps[x] = pack_read(my_txt, st[x]);
          lm[x] = s_lenmask[wl[x] - 1 < 16u ? wl[x] : 1u];
        }
#pragma unroll
        for (int x = 0; x < NX; ++x) {
          pin(ps[x]);
          pin(lm[x]);
        }
#pragma unroll
        for (int x = 0; x < NX; ++x) doc[x] = nb == 0 ? (rb < 0 ? 0u : (uint32_t)rb) : doc_at(st[x]);
#pragma unroll
        for (int x = 0; x < NX; ++x) {
          uint64_t lo, hi;
          pack_join(ps[x], lm[x], &lo, &hi);
          key[x] = key4(lo, hi);
          key[x].z |= spread4(doc[x] & 15u);
          key[x].w |= spread4(doc[x] >> 4);
          h[x] = red_hash(key[x]);
        }
#pragma unroll
        for (int x = 0; x < NX; ++x)
          if (in[x] && wl[x] - 1 >= 16u) {
            key[x] = with_doc(long_word(st[x], wl[x], doc[x]), doc[x]);
            h[x] = place_hash(key[x]);
            wait_vmem();
          }
        const int res = table_add<NX, true>(T, key, h, one, in, left, spare);
        if (res == kNoRoom) spill(key, left, nx);
        else if (res == kNoSlot && lane == 0) or32(&hdr_of()->flags, kFlagStall);
      };
      for (uint32_t w0 = 0; w0 < n; w0 += kList) {
        list_starts(start16, lane * 16, incl - c - w0, n <= kList, kList, my_starts);
        wave_sync();
        // two tokens a lane while more than 64 are left, then one
        const uint32_t nl = min(n - w0, kList);
        uint32_t at = 0;
        for (; at + 64 < nl; at += 128) count(std::integral_constant<int, 2>(), at, nl - at);
        if (at < nl) count(std::integral_constant<int, 1>(), at, nl - at);
        wave_sync();
      }
      k = kn;
    }
  };

  // ---- places of entries inside their documents ---------------------------------------------
  // (entries << 32 | bytes) before this lane's entry in document r; called by whole waves. The
  // lanes of one document, the common case, take their places with one LDS atomic.
  auto place = [&](bool valid, uint32_t r, uint32_t wl) -> uint64_t {
    const uint64_t m = __ballot(valid);
    if (m == 0) return 0;
    const uint32_t r0 = (uint32_t)__builtin_amdgcn_readlane((int)r, (int)(__ffsll((unsigned long long)m) - 1));
    if (__all(!valid || r == r0)) {
      const uint32_t incl = wave_incl_scan(valid ? wl : 0u);
      const uint32_t tot = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
      uint64_t b = 0;
      if (lane == 0) b = atomicAdd(&s_dcur[r0], ((unsigned long long)__popcll(m) << 32) | tot);
      const uint32_t be = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32));
      const uint32_t bb = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b);
      const uint32_t i = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
      return ((uint64_t)(be + i) << 32) | (bb + incl - (valid ? wl : 0u));
    }
    return valid ? atomicAdd(&s_dcur[r], (1ull << 32) | wl) : 0ull;
  };

  // Tables set aside: a chain of a header slot (the one before it, entries) and a slot per entry
  // (key, count, place).
  uint32_t dump = 0;
  // (all threads, after a barrier; ends with one, the table empty)
  auto set_aside = [&]() {
    const uint32_t ne = min(s_nent, T.cap);
    if (tid == 0) {
      s_at = take(ne + 1);
      if (!s_lost) *slot_at(s_at) = Slot{dump, ne, 0, 0};
    }
    __syncthreads();
    const uint32_t d = s_at;
    const bool ok = !s_lost;
    for (uint32_t i0 = 0; i0 < ne; i0 += kBlk) {
      const uint32_t i = i0 + tid;
      const uint32_t cnt = i < ne ? T.cnt[i] : 0u;
      const uint4 k = i < ne ? T.key[i] : make_uint4(0, 0, 0, 0);
      const uint64_t at = place(cnt != 0, key_doc(k), (uint32_t)key_len(without_doc(k)));
      if (ok && i < ne)
        *slot_at(d + 1 + i) = Slot{(uint64_t)k.x | ((uint64_t)k.y << 32), cnt, (uint64_t)k.z | ((uint64_t)k.w << 32), at};
    }
    if (ok) dump = d + 1;
    __syncthreads();
    for (uint32_t i = tid; i < kDocSlots / 4; i += kBlk) ((uint4*)T.slot)[i] = make_uint4(0, 0, 0, 0);
    if (tid == 0) s_nent = 0;
    __syncthreads();
  };
  // the records of this wave's chain: f(record, present), 64 at a time
  auto each_spilled = [&](auto f) {
    for (uint32_t cu = chunk; cu;) {
      uint4* const rec = (uint4*)slot_at(cu - 1);
      const uint32_t n = cu == chunk ? chunk_n : kChunkRecs;
      for (uint32_t i = 0; i < n; i += 64) f(rec + 1 + i + lane, i + lane < n);
      cu = rec[0].x;
    }
  };
  auto part_of = [&](uint32_t h, uint32_t level) -> uint32_t { return mix32(h + level * 0x9e3779b9u) >> 24; };
  // spilled keys that have an entry are counted; those left are counted by part
  auto settle = [&](uint32_t level) {
    each_spilled([&](uint4* rec, bool in) {
      if (!in) return;
      const uint4 k = *rec;
      if ((k.x | k.y | k.z | k.w) == 0) return;
      const uint32_t h = place_hash(k);
      const int at = table_find(T, k, h);
      if (at >= 0) {
        lds_add(&T.cnt[at], 1u);
        *rec = make_uint4(0, 0, 0, 0);
      } else {
        atomicAdd(&s_part[part_of(h, level)], 1u);
      }
    });
  };
  // The keys rec(j), j < n, are counted by all waves.
  auto insert = [&](uint32_t n, auto rec) {
    const uint32_t one[2] = {1u, 1u};
    for (uint32_t i = wv * 128; i < n; i += kWaves * 128) {
      uint4 k[2];
      uint32_t h[2];
      bool use[2], left[2];
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        const uint32_t j = i + 64 * x + lane;
        use[x] = j < n;
        k[x] = use[x] ? *rec(j) : make_uint4(0, 0, 0, 0);
        h[x] = place_hash(k[x]);
      }
      const int res = table_add<2, true>(T, k, h, one, use, left);
      if (res == kNoRoom) spill(k, left, std::integral_constant<int, 2>());
      else if (res == kNoSlot && lane == 0) or32(&hdr_of()->flags, kFlagStall);
    }
  };
  // One level of the spilled keys (all threads, after a barrier; ends with one).
  auto count_spilled = [&](uint32_t level) {
    if (tid < kDocParts) s_part[tid] = 0;
    __syncthreads();
    settle(level);
    __syncthreads();
    set_aside();
    // parts' places among the keys left, which are copied in their order
    uint32_t v = 0, incl = 0;
    if (tid < kDocParts) {
      v = s_part[tid];
      incl = wave_incl_scan(v);
      if (lane == 63) s_sum[wv] = incl;
    }
    __syncthreads();
    const uint32_t S = (uint32_t)(s_sum[0] + s_sum[1] + s_sum[2] + s_sum[3]);
    if (tid < kDocParts) {
      for (uint32_t w = 0; w < wv; ++w) incl += (uint32_t)s_sum[w];
      s_part[tid] = incl - v;
    }
    if (tid == 0) {
      s_spill = 0;
      if (S) s_at = take((S + 1) / 2);
    }
    __syncthreads();
    if (S == 0 || s_lost) return;
    const uint32_t base = s_at;
    auto copy_at = [&](uint32_t j) -> uint4* { return (uint4*)slot_at(base + j / 2) + (j & 1); };
    each_spilled([&](uint4* rec, bool in) {
      if (!in) return;
      const uint4 k = *rec;
      if ((k.x | k.y | k.z | k.w) != 0)
        *copy_at(atomicAdd(&s_part[part_of(place_hash(k), level)], 1u)) = k;
    });
    chunk = 0;
    chunk_n = 0;
    __syncthreads();
    // s_part[p] is now the end of part p
    for (uint32_t p = 0; p < kDocParts;) {
      const uint32_t a = p ? s_part[p - 1] : 0u, room = T.cap - min(s_nent, T.cap);
      uint32_t e = p;
      while (e < kDocParts && s_part[e] - a <= room) ++e;
      if (e == p) {
        if (s_nent) {
          __syncthreads();
          set_aside();
          continue;
        }
        ++e;  // too many keys for any table: some may spill
      }
      const uint32_t n = s_part[e - 1] - a;
      __syncthreads();
      insert(n, [&](uint32_t j) { return copy_at(a + j); });
      __syncthreads();
      if (n > T.cap && s_spill && !s_lost) {
        // (the histogram of this call is thrown away: the parts' ends stay)
        each_spilled([&](uint4* rec, bool in) {
          if (!in) return;
          const uint4 k = *rec;
          const int at = (k.x | k.y | k.z | k.w) ? table_find(T, k, place_hash(k)) : -1;
          if (at >= 0) {
            lds_add(&T.cnt[at], 1u);
            *rec = make_uint4(0, 0, 0, 0);
          }
        });
        __syncthreads();
      }
      if (s_lost) break;
      p = e;
    }
    __syncthreads();
  };

  struct Out {
    uint64_t *woff, *docs, bias;
    uint8_t* words;
    void* counts;
    uint32_t count_bytes;
  };
  auto put = [&](const Out& o, uint64_t e, uint64_t b, const uint4 k, uint64_t cnt, uint64_t d) {
    o.woff[e] = b;
    // a document has fewer than 2^31 tokens (the corpus is below 4 GiB), so only a debug bias can
    // take a count past the 32-bit width
    const uint64_t c = cnt + o.bias;
    if (o.count_bytes == 4) {
      if (c > 0x7fffffffull) or32(&hdr_of()->flags, kFlagCountOverflow);
      ((int32_t*)o.counts)[e] = (int32_t)c;
    } else {
      ((int64_t*)o.counts)[e] = (int64_t)c;
    }
    o.docs[e] = d;
    if (is_long_key(k)) {
      store_long(o.words + b, long_ptr(k), k.z);
    } else {
      store_word(o.words + b, (uint64_t)k.x | ((uint64_t)k.y << 32), (uint64_t)k.z | ((uint64_t)k.w << 32),
                 (uint32_t)key_len(k));
    }
  };

  // ---- the queue ------------------------------------------------------------------------------
  // An item is a run of documents, 0 when there is none left. The
  // queue takes them by size class, the largest first (a workgroup that took a large document
  // late would otherwise finish alone).
  if (tid == 0) {
    uint32_t n = 0;
    for (int k = kDocClasses - 1; k >= 0; --k) {
      s_class[kDocClasses - 1 - k] = n;
      n += as_global(args()->class_n)[k];
    }
    s_class[kDocClasses] = n;
  }
  __syncthreads();
  auto item_at = [&](uint32_t q) -> uint64_t {
    if (q >= s_class[kDocClasses]) return 0;
    const uint32_t at = s_class[min(lane, kDocClasses - 1)];
    const uint32_t c = 31 - (uint32_t)__clz((int)(uint32_t)(__ballot(at <= q) & ((1u << kDocClasses) - 1)));
    const uint32_t i = q - (uint32_t)__builtin_amdgcn_readlane((int)at, (int)c);
    return uniform64(as_global(args()->items)[args()->class_at[kDocClasses - 1 - c] + i]);
  };
  auto next_pos = [&]() -> uint32_t {  // (one lane's)
    return gridDim.x + (uint32_t)atomicAdd((unsigned long long*)&hdr_of()->work_next, 1ull);
  };
  uint32_t lost_most = 0;
  if (tid == 0) {
    s_tokens = 0;
    s_nent = s_spill = s_used = s_done = 0;
    s_tile = kWaves;
    s_next = next_pos();
  }
  uint64_t it = item_at(blockIdx.x);
  uint32_t cur = 0;  // s_doff buffer of the group
  if (it && tid <= item_docs(it)) s_doff[0][tid] = offset_at(item_first(it) + tid);
  __syncthreads();
  uint64_t ahead = item_at(s_next);
  if (ahead && tid <= item_docs(ahead)) s_doff[1][tid] = offset_at(item_first(ahead) + tid);
  __syncthreads();
  if (it) t0 = load((int64_t)uniform64(s_doff[0][0]), (int64_t)uniform64(s_doff[0][item_docs(it)]), wv);
  while (it) {
    const uint32_t nd = item_docs(it);
    const uint64_t d0 = item_first(it);
    const uint64_t* const doff = s_doff[cur];
    chunk = 0;
    chunk_n = 0;
    dump = 0;
    scan(doff, nd);
    // the first wave that is done takes the position after the next (asked for by wave 0 before
    // the scan, its answer was waited for on the spot, with the acknowledgements of the stores of
    // the group before: 20 % of the time)
    if (lane == 0 && atomicAdd(&s_done, 1u) == 0) s_next = next_pos();
    __syncthreads();
    const uint64_t after = ahead ? item_at(s_next) : 0;
    const uint32_t nxt = cur == 2 ? 0 : cur + 1, nxt2 = cur == 0 ? 2 : cur - 1;
    if (ahead) t0 = load((int64_t)uniform64(s_doff[nxt][0]), (int64_t)uniform64(s_doff[nxt][item_docs(ahead)]), wv);
    if (s_spill) {
      if (tid == 0) add64(&hdr_of()->stat[3], nd);
      for (uint32_t level = 0; s_spill && !s_lost; ++level) count_spilled(level);
      if (s_lost && tid == 0 && s_used > lost_most) {  // what the rest would have taken, roughly
        add64(&hdr_of()->arena_next, 3ull * (s_used - lost_most));
        lost_most = s_used;
      }
    }
    // places of the entries in their documents; the slots are not needed any more
    clear_slots();
    const uint32_t ne = min(s_nent, T.cap);
    uint64_t at[kPerThread];
#pragma unroll
    for (uint32_t x = 0; x < kPerThread; ++x) {
      const uint32_t i = tid + x * kBlk;
      at[x] = 0;
      if (x * kBlk < ne) {
        const uint32_t cnt = i < ne ? T.cnt[i] : 0u;
        const uint4 k = i < ne ? T.key[i] : make_uint4(0, 0, 0, 0);
        at[x] = place(cnt != 0, key_doc(k), (uint32_t)key_len(without_doc(k)));
      }
    }
    uint64_t off = 0;
    if (after && tid <= item_docs(after)) off = offset_at(item_first(after) + tid);
    __syncthreads();
    // documents' places in the group, and its place in the output, by wave 0; the other waves
    // go on to their text of the next group
    if (wv == 0) {
      uint64_t v[kDocW / 64], incl = 0;
#pragma unroll
      for (uint32_t j = 0; j < kDocW / 64; ++j) {
        const uint32_t r = lane * (kDocW / 64) + j;
        v[j] = r < nd ? s_dcur[r] : 0ull;
        incl += v[j];
      }
      const uint64_t sum = incl;
      const uint32_t ie = wave_incl_scan((uint32_t)(sum >> 32)), ib = wave_incl_scan((uint32_t)sum);
      incl = ((uint64_t)ie << 32) | ib;
      uint64_t o = 0;
      if (lane == 63) o = atomicAdd((unsigned long long*)&hdr_of()->out_cursor, (unsigned long long)incl);
      o = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(o >> 32), 63) << 32) |
          (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)o, 63);
      uint64_t first = o + incl - sum;
#pragma unroll
      for (uint32_t j = 0; j < kDocW / 64; ++j) {
        const uint32_t r = lane * (kDocW / 64) + j;
        if (r < nd) {
          s_dcur[r] = first;
          as_global(args()->doc_ptr)[d0 + r] = first >> 32;
          as_global(args()->doc_len)[d0 + r] = v[j] >> 32;
        }
        first += v[j];
      }
      if (lane == 63) {
        s_out = first;  // the end of the group's output
        s_nent = s_spill = s_used = s_done = 0;
        s_tile = kWaves;
        if ((first >> 32) > args()->cap_e || (first & 0xffffffffull) > args()->cap_b) or32(&hdr_of()->flags, kFlagWordCap);
      }
    }
    // what was asked for before the entries' stores is taken before them (loads and stores are
    // waited for in their order)
    if (after && tid <= item_docs(after)) s_doff[nxt2][tid] = off;
    pin(t0);
    __syncthreads();
    const bool room = (s_out >> 32) <= args()->cap_e && (s_out & 0xffffffffull) <= args()->cap_b;
    if (room) {
      const Args A = args();
      const Out o{as_global(A->word_offsets), as_global(A->docs), A->count_bias, as_global(A->words),
                  (void*)as_global((uint8_t*)A->counts), A->count_bytes};
#pragma unroll
      for (uint32_t x = 0; x < kPerThread; ++x) {
        const uint32_t i = tid + x * kBlk;
        if (i >= ne) continue;
        const uint32_t cnt = T.cnt[i];
        if (!cnt) continue;
        const uint4 k = T.key[i];
        const uint32_t r = key_doc(k);
        const uint64_t pos = s_dcur[r] + at[x];
        put(o, pos >> 32, pos & 0xffffffffull, without_doc(k), cnt, d0 + r);
      }
      for (uint32_t du = s_lost ? 0u : dump; du;) {
        const Slot h = *slot_at(du - 1);
        for (uint32_t i = tid; i < (uint32_t)h.cnt; i += kBlk) {
          const Slot sl = *slot_at(du + i);
          if (!sl.cnt) continue;
          const uint4 k = key4(sl.key, sl.w0);
          const uint32_t r = key_doc(k);
          const uint64_t pos = s_dcur[r] + sl.w1;
          put(o, pos >> 32, pos & 0xffffffffull, without_doc(k), sl.cnt, d0 + r);
        }
        du = (uint32_t)h.key;
      }
    }
    __syncthreads();  // the table and the places are free again
    for (uint32_t r = tid; r < nd; r += kBlk) s_dcur[r] = 0;
    it = ahead;
    ahead = after;
    cur = nxt;
  }
  if (lane == 0 && tokens) atomicAdd(&s_tokens, (unsigned long long)tokens);
  __syncthreads();
  if (tid == 0) {
    if (s_tokens) add64(&hdr_of()->total_tokens, s_tokens);
    // (the cursor, which the last workgroup reads, has answered all of this one's additions)
    const uint64_t done = __hip_atomic_fetch_add(&hdr_of()->occupied, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (done + 1 == gridDim.x) {  // the last workgroup closes the output
      const uint64_t c = ld_relaxed(&hdr_of()->out_cursor);
      hdr_of()->n_entries = c >> 32;
      hdr_of()->word_bytes = c & 0xffffffffull;
      if ((c >> 32) <= args()->cap_e) as_global(args()->word_offsets)[c >> 32] = c & 0xffffffffull;
    }
  }
}

// Bytes per work item where the caller has not said: the fewest items that are the same number for
// every workgroup and at most kMaxWin bytes. Fewer and larger ones have less to wait for between
// them (the output's place, the first text; about 5 us an item), until many do not fit the table:
// kernel time of 100,000 documents (2.7 GB) with 16 / 24 / 32 / 48 / 64 KiB 8.4 / 8.3 / 7.5 / 7.1 /
// 7.6 ms. With few to a workgroup some would take one more than others: 2,000 documents (17.6 MB,
// 256 workgroups) took 94 us with 32 KiB, 2.1 items each, and 81 with 34, two each.
WC_DEV uint64_t window_bytes(uint64_t len, uint32_t grid) {
  const uint64_t k = (len + grid * kMaxWin - 1) / (grid * kMaxWin);  // items per workgroup
  const uint64_t w = (len + grid * max(k, (uint64_t)1) - 1) / (grid * max(k, (uint64_t)1));
  return min(max((w + 1023) & ~1023ull, kMinWin), kMaxWin);
}

__global__ void doc_begin_kernel(Header* hdr, DocTask* task, DocTask value) {
  if (threadIdx.x < kDocHeadBytes / 4) ((uint32_t*)hdr)[threadIdx.x] = 0;
  if (threadIdx.x == 0) *task = value;
}

// Checks the offsets and lists the work items in their size classes: documents longer than a window
// by themselves, and the rest of each window's documents, by the thread of the first of them. (More
// than kDocW documents: several items, in class 0.) Items are ranked in LDS, and a workgroup takes
// its places with an atomic per class: one per wave and class, on few addresses, took 98 us for
// 100,000 documents instead of 25.
__global__ __launch_bounds__(kBlk) void doc_plan_kernel(DocParams P) {
  __shared__ uint32_t s_n[kDocClasses], s_at[kDocClasses];
  const uint64_t len = P.task->len, n_docs = P.task->n_docs;
  const uint64_t* offsets = as_global(P.task->offsets);
  const uint32_t lane = threadIdx.x & 63;
  const uint64_t step = (uint64_t)gridDim.x * blockDim.x;
  const uint64_t win = P.win_bytes ? P.win_bytes : window_bytes(len, P.grid);
  const uint64_t limit = P.direct_kib ? max(win, (uint64_t)P.direct_kib << 10) : ~0ull;
  for (uint64_t i0 = blockIdx.x * (uint64_t)blockDim.x; i0 <= n_docs; i0 += step) {
    const uint64_t i = i0 + threadIdx.x;
    if (threadIdx.x < kDocClasses) s_n[threadIdx.x] = 0;
    __syncthreads();
    const uint64_t a = i <= n_docs ? offsets[i] : 0, b = i < n_docs ? offsets[i + 1] : a;
    const bool bad = i <= n_docs && (a > b || (i == n_docs && a > len));
    if (bad) or32(&P.hdr->flags, kFlagBadOffsets);
    const bool doc = i < n_docs && !bad;
    const bool alone = doc && b - a > win;
    const uint64_t over = __ballot(doc && b - a > limit);
    if (over && lane == 0) add64(&P.hdr->over_n, (uint64_t)__popcll(over));
    uint64_t end = i;  // documents [i, end) of this lane's window
    if (doc && b - a <= win && (i == 0 || offsets[i - 1] / win != a / win)) {
      const uint64_t x = (a / win + 1) * win;
      uint64_t lo = i + 1, hi = lo, s = 1;  // offsets[lo - 1] < x
      while (hi < n_docs && offsets[hi] < x) {
        lo = hi + 1;
        hi = min(hi + s, n_docs);
        s *= 2;
      }
      while (lo < hi) {
        const uint64_t mid = (lo + hi) >> 1;
        if (offsets[mid] < x) lo = mid + 1; else hi = mid;
      }
      end = lo;
      const uint64_t z = offsets[end] - offsets[end - 1];
      if (end - 1 > i && z > win && z <= len) --end;  // the window's last, listed by its own lane
    }
    if (alone) end = i + 1;
    const uint32_t n = (uint32_t)((end - i + kDocW - 1) / kDocW);
    uint32_t cls = 0;
    if (n == 1) {
      const uint64_t bytes = offsets[end] - a;
      cls = bytes < (16u << 10) ? 0u : min(63u - (uint32_t)__clzll((long long)(bytes >> 13)), kDocClasses - 1);
    }
    uint32_t at = n ? atomicAdd(&s_n[cls], n) : 0u;
    __syncthreads();
    if (threadIdx.x < kDocClasses && s_n[threadIdx.x])
      s_at[threadIdx.x] = atomicAdd(&P.class_n[threadIdx.x], s_n[threadIdx.x]);
    __syncthreads();
    if (n) {
      at += s_at[cls];
      // (runs of offsets in order fit their class; others fail the call)
      const uint64_t lo = P.class_at[cls], hi = P.class_at[cls + 1];
      for (uint64_t d = i; d < end; d += kDocW, ++at)
        if (lo + at < hi) P.items[lo + at] = (min((uint64_t)kDocW, end - d) << kItemShift) | d;
    }
    __syncthreads();
  }
}

hipError_t set_doc_smem() {
  return hipFuncSetAttribute((const void*)doc_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kDyn);
}

hipError_t launch_doc_begin(Header* hdr, DocTask* task, const DocTask& value, hipStream_t s) {
  hipLaunchKernelGGL(doc_begin_kernel, dim3(1), dim3(64), 0, s, hdr, task, value);
  return hipGetLastError();
}

hipError_t launch_docs(const DocParams& P, hipStream_t s) {
  hipLaunchKernelGGL(doc_plan_kernel, dim3(256), dim3(kBlk), 0, s, P);
  hipLaunchKernelGGL(doc_kernel, dim3(P.grid), dim3(kBlk), kDyn, s, P);
  return hipGetLastError();
}

}  // namespace wc
