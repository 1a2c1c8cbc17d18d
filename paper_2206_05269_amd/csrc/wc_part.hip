// Partitioned global count, for texts up to the size from which the two-pass count with a sampled
// dictionary (wc_global.hip) pays: the map of Section 3 (tokenise, count) in LDS, and the reduce
// (sum the counts of each word) over hash partitions, each of which leaves LDS straight into the
// result arrays. There is no table in device memory: nothing to clear, no device atomic per
// word and no compaction pass.
//
//   part_map_kernel: each workgroup scans a contiguous range of the text and counts its words in
//     an LDS table. When the table is nearly full, and at the end of the range, its words leave
//     as a list of (word, count) records ordered by partition, with the place of every partition
//     in a directory.
//   part_reduce_kernel: one workgroup per partition adds the partition's records of every list
//     in an LDS table and writes each distinct word, its count and its bytes to the output.
//
// A text of at most kSingleBytes is counted and written by one workgroup in one launch.
//
// Why. The one-pass kernel (wc_count.hip) keeps 2,048 words per workgroup and adds them to one
// device table at every flush: on a 20 MB text of 50,000 words that is about 2.6 million inserts,
// many of them on the same few hot slots (381 us, 52 GB/s); clearing and compacting the table took
// another 65 us. Here a word costs one 20-byte record per list it occurs in, written and read once,
// and contention stays in LDS.
//
// Words longer than 16 bytes are kept as references to an occurrence and compared by content.
// What does not fit (more records than the arena, more lists than the directory) sets kFlagArena,
// more long words alike in length and hash than a table holds set kFlagSplit, and the caller counts
// the text again with the one-pass kernel.
#include <type_traits>

#include "wc_internal.h"
#include "wc_stripe.h"
#include "wc_utf8.h"
#include "wc_words.h"

namespace wc {

namespace {

constexpr int kBlk = 1024;
constexpr uint32_t kWaves = kBlk / 64;
constexpr uint32_t kText = kStripe + 32;     // per wave: a tile with the bytes around it, padding
constexpr uint32_t kList = 192;              // starts of a tile listed at a time
constexpr uint32_t kEnds = kStripe / 32 + 2; // word-end bitmap of the staged text, two words of zeros
constexpr uint32_t kListWords = kList / 2 + kEnds;

constexpr uint32_t kPerThread = (kPartMapEntries + kBlk - 1) / kBlk;

// Exclusive sums over the workgroup of a pair packed in 64 bits (no field overflows).
WC_DEV uint64_t block_scan64(uint64_t v, uint64_t* s_tmp, uint64_t* total) {
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint64_t incl = v;
  for (int d = 1; d < 64; d <<= 1) {
    const uint64_t y = __shfl_up(incl, d, 64);
    if (lane >= (uint32_t)d) incl += y;
  }
  if (lane == 63) s_tmp[wave] = incl;
  __syncthreads();
  uint64_t base = 0, tot = 0;
  for (uint32_t w = 0; w < kWaves; ++w) {
    const uint64_t x = s_tmp[w];
    base += w < wave ? x : 0;
    tot += x;
  }
  __syncthreads();
  *total = tot;
  return base + incl - v;
}

// The output cursor. Counting a text (below 2^28 bytes): partitions done << 55 | entries << 28 |
// word bytes, so that one atomic reserves a partition's space and tells the last one that it is
// the last. Merging tables (wide, below 2^32 entries and word bytes): entries << 32 | bytes, and the
// partitions done are counted beside it.
constexpr uint32_t kCurPart = 55;
WC_DEV uint64_t cur_entries(uint64_t c, bool wide) {
  return wide ? c >> 32 : (c >> 28) & ((1ull << (kCurPart - 28)) - 1);
}
WC_DEV uint64_t cur_bytes(uint64_t c, bool wide) { return c & (wide ? 0xffffffffull : 0xfffffffull); }

// Totals and limits, once every entry has its place (one thread).
WC_DEV void finish_output(const PartParams& P, uint64_t n, uint64_t b) {
  P.hdr->n_entries = n;
  P.hdr->word_bytes = b;
  if (n <= P.slots) P.word_offsets[n] = b;
  if (n > P.occ_limit) or32(&P.hdr->flags, kFlagTableFull);
  if (b > P.word_cap) or32(&P.hdr->flags, kFlagWordCap);
}

// Every entry of the table with a count to the output arrays; `last`: nothing of this partition
// comes after. All threads.
template <bool kWide, class C>
WC_DEV void export_table(const PartParams& P, const PartTable<C>& T, bool last, uint32_t parts,
                         uint64_t* s_tmp, uint64_t* s_base) {
  const uint32_t tid = threadIdx.x, ne = min(*T.n, T.cap);
  uint64_t part = 0;  // entries << 32 | bytes
  for (uint32_t i = tid; i < ne; i += kBlk)
    if (T.cnt[i]) part += (1ull << 32) + key_len(T.key[i]);
  uint64_t tot;
  const uint64_t at = block_scan64(part, s_tmp, &tot);
  if (tid == 0) {
    const uint64_t tn = tot >> 32, tb = tot & 0xffffffffull;
    unsigned long long* const cur = (unsigned long long*)&P.hdr->out_cursor;
    if (kWide) {
      *s_base = atomicAdd(cur, (unsigned long long)tot);
    } else {
      const uint64_t add = (last ? 1ull << kCurPart : 0ull) | (tn << 28) | tb;
      *s_base = atomicAdd(cur, (unsigned long long)add);
      const uint64_t now = *s_base + add;
      if (last && now >> kCurPart == parts) finish_output(P, cur_entries(now, false), cur_bytes(now, false));
    }
  }
  __syncthreads();
  uint64_t e = cur_entries(*s_base, kWide) + (at >> 32);
  uint64_t b = cur_bytes(*s_base, kWide) + (at & 0xffffffffull);
  for (uint32_t i = tid; i < ne; i += kBlk) {
    const C n = T.cnt[i];
    if (!n) continue;
    const uint4 k = T.key[i];
    const uint64_t len = key_len(k);
    if (e < P.slots) {  // beyond: the call fails as full
      const uint64_t c = (uint64_t)n + P.count_bias;
      P.word_offsets[e] = b;
      if (P.count_bytes == 4) {
        if (c > 0x7fffffffull) or32(&P.hdr->flags, kFlagCountOverflow);
        ((int32_t*)P.counts)[e] = (int32_t)c;
      } else {
        ((int64_t*)P.counts)[e] = (int64_t)c;
      }
    }
    if (b + len <= P.word_cap) {
      if (is_long_key(k)) {
        store_long(P.words + b, long_ptr(k), len);
      } else {
        store_word(P.words + b, (uint64_t)k.x | ((uint64_t)k.y << 32),
                   (uint64_t)k.z | ((uint64_t)k.w << 32), (uint32_t)len);
      }
    }
    ++e;
    b += len;
  }
  __syncthreads();
  if (kWide && last && tid == 0) {
    // (what the last one reads, the cursor, has answered this workgroup's addition: no fence, which
    // writes the XCD's L2 back, before this one: reduce of 2,000 tables 26 -> 23 us)
    const uint64_t done = __hip_atomic_fetch_add(&P.hdr->work_next, 1ull, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT);
    if (done + 1 == parts) {
      const uint64_t c = ld_relaxed(&P.hdr->out_cursor);
      finish_output(P, cur_entries(c, true), cur_bytes(c, true));
    }
  }
}

}  // namespace

// ---------------------------------------------------------------------------------------
// map
// ---------------------------------------------------------------------------------------
// The workgroup's range is cut into tiles of 992 bytes, staged with the 16 bytes before and after
// them, so a word of at most 16 bytes is read whole from LDS; a longer one from device memory. A wave
// that has counted a tile takes the next one that is left; waves meet only when the table is to be
// emptied. (With equal runs of 1 KiB stripes, their next one classified a
// step early, the last waves were alone at the end: map of 20 MB 50 -> 43 us, of 64 MB 166 -> 141.)
//
// Bound by instructions (a 64 MB text: 473 GB/s of text, 724 vector and 490 scalar instructions per
// KiB, the vector units busy for 61 % of the time). What the scan does not use stays out of its registers, and the rest of
// a tile's words after the first 128 is counted one a lane: map of 20 MB 56 -> 51 us, of 64 MB
// 186 -> 170.
//
// UTF-8. A tile is staged with 32 bytes after it, so that the sequences are whole in all 16 bytes
// that a short word can reach. ASCII text takes the same steps as without UTF-8, and one test per
// tile.
template <bool kSingle, bool kUtf8>
__global__ __launch_bounds__(kBlk) void part_map_kernel(PartParams P) {
  // What the scan does not need is read with args(): by name it would be loaded once, at the start,
  // and held or spilled over the scan.
  typedef const __attribute__((address_space(4))) PartParams* Args;
  auto args = []() -> Args {
    Args a = (Args)__builtin_amdgcn_kernarg_segment_ptr();
    __asm__ volatile("" : "+s"(a));
    return a;
  };
  extern __shared__ __align__(16) uint8_t s_dyn[];
  __shared__ uint32_t s_list[kWaves][kListWords];  // starts (16 bits each), then the end bitmap
  __shared__ uint32_t s_bnd[kWaves][kEnds];
  __shared__ uint4 s_lenmask[17];
  __shared__ uint32_t s_hist[kParts], s_start[kParts];
  __shared__ uint32_t s_nent, s_done, s_tokens, s_tile, s_scan[4];
  __shared__ uint64_t s_tmp[kWaves], s_base;
  PartTable<uint32_t> T;
  T.slot = (uint32_t*)s_dyn;
  T.key = (uint4*)(T.slot + kRedSlots);
  T.cnt = (uint32_t*)(T.key + kPartMapEntries);
  T.n = &s_nent;
  T.cap = kPartMapEntries;
  const uint32_t tid = threadIdx.x, lane = tid & 63;
  const uint32_t wv = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
  uint8_t* const my_txt = (uint8_t*)(T.cnt + kPartMapEntries) + wv * kText;
  uint16_t* const my_starts = (uint16_t*)s_list[wv];
  uint32_t* const my_ends = s_list[wv] + kList / 2;
  uint32_t* const my_bnd = s_bnd[wv];
  auto hdr_of = [&]() -> Header* { return as_global(args()->hdr); };

  // The workgroup's text [G0, G1) in tiles of kTile bytes, staged with the 16 bytes before them and
  // the 16 (UTF-8: 32) after: a lane reads 16 bytes. Bytes outside the text may be anything.
  constexpr uint32_t kTile = kStripe - (kUtf8 ? 48 : 32);
  const uint64_t first = (uint64_t)blockIdx.x * P.stripes_per_wg;
  const int64_t G0 = P.base_off + (int64_t)(first * kStripe);
  const int64_t G1 = P.base_off + (int64_t)(min(first + P.stripes_per_wg, P.n_stripes) * kStripe);
  auto tile_at = [&](uint32_t k) -> int64_t { return G0 + (int64_t)((uint64_t)k * kTile); };
  auto load = [&](uint32_t k) -> uint4 {
    const int64_t p = tile_at(k) - 16;
    uint4 v = make_uint4(0x20202020u, 0x20202020u, 0x20202020u, 0x20202020u);
    if (p + 16 >= G1) return v;
    uint32_t at = lane * 16;
    pin(at);  // (an offset to a scalar address: as a sum of its own it was kept, and spilled)
    if (p >= 0 && p + (int64_t)kStripe <= (int64_t)P.len) v = load_stream16(P.corpus + p + at);
    else v = load_text16(P.corpus, P.len, p + at);
    return v;
  };
  uint32_t kn = wv;  // the wave's next tile, its bytes in raw
  uint4 raw = load(kn);

  for (uint32_t i = tid; i < kRedSlots / 4; i += kBlk) ((uint4*)T.slot)[i] = make_uint4(0, 0, 0, 0);
  for (uint32_t i = tid; i < kWaves * kListWords; i += kBlk) (&s_list[0][0])[i] = 0;
  for (uint32_t i = tid; i < kWaves * kEnds; i += kBlk) (&s_bnd[0][0])[i] = 0;
  if (tid < kParts) s_hist[tid] = 0;
  init_len_masks(s_lenmask, tid, kBlk);
  if (tid == 0) {
    s_nent = 0;
    s_done = 0;
    s_tokens = 0;
    s_tile = kWaves;
    if (kSingle) {
      *hdr_of() = Header{};
      __threadfence();
    }
  }
  __syncthreads();

  // Offsets must be non-decreasing and end inside the text; a bad one fails the call. Until the
  // host sees that, positions taken from them are only compared, and ranges are cut to the text.
  for (uint64_t d = blockIdx.x * (uint64_t)kBlk + tid; d <= P.n_docs; d += (uint64_t)gridDim.x * kBlk) {
    const uint64_t o = P.offsets[d];
    if (d < P.n_docs ? o > P.offsets[d + 1] : o > P.len) or32(&hdr_of()->flags, kFlagBadOffsets);
  }
  const int64_t R0 = (int64_t)min(P.offsets[0], P.len), R1 = (int64_t)min(P.offsets[P.n_docs], P.len);

  // Document starts, 64 at a time in the lanes (lane l: document d0 + l): all documents before d0
  // start before the tile at hand.
  uint64_t d0 = 0;
  int64_t doff;
  auto start_of = [&](uint64_t d) -> int64_t {
    return d <= P.n_docs ? (int64_t)P.offsets[d] : INT64_MAX;
  };
  auto first_from = [&](int64_t p, uint64_t lo) -> uint64_t {  // 64 probes at a time
    uint64_t hi = P.n_docs + 1;  // offsets[lo - 1] < p <= offsets[hi]
    while (hi > lo && hi - lo > 64) {
      const uint64_t step = (hi - lo + 63) / 64, d = lo + lane * step;
      const uint64_t m = __ballot(d < hi && start_of(d) < p);
      const uint64_t k = (uint64_t)__popcll(m);
      if (k == 0) {
        hi = lo;
      } else {
        hi = min(hi, lo + k * step);
        lo += (k - 1) * step + 1;
      }
    }
    return lo;
  };
  auto seek = [&](int64_t p, uint64_t lo) {
    d0 = first_from(p, lo);
    doff = start_of(d0 + lane);
  };
  seek(tile_at(kn) - 16, 0);
  auto doc_limit = [&](uint64_t pos) -> uint64_t {  // first document start after pos, or the end
    const uint64_t* const offsets = as_global(args()->offsets);
    uint64_t a = 1, b = args()->n_docs;
    while (a < b) {
      const uint64_t m = (a + b) >> 1;
      if (offsets[m] > pos) b = m;
      else a = m + 1;
    }
    return min(offsets[a], P.len);
  };

  bool done = false, counted = false;  // no tiles are left
  uint32_t n = 0, w0 = 0, off = 0, start16 = 0, rank = 0;  // off: place of token w0 in the list
  int64_t p0 = 0;
  uint32_t tokens = 0;
  bool over = false;  // a word found no room (this lane)

  // Key of the word at staged byte s, longer than 16 bytes; len: its length, or 0 when its end is
  // not within 32 bytes. Its bytes come from the staged text when its end is staged.
  auto long_word = [&](uint32_t s, uint32_t len) -> uint4 {
    const uint8_t* const p = P.corpus + (p0 + s);
    for (uint32_t w = (s + 32) >> 5; !len && w < kEnds; ++w) {
      uint32_t m = my_ends[w];
      if (w == (s + 32) >> 5) m &= 0xffffffffu << (s & 31);
      if (m) len = w * 32 + __ffs(m) - s;
    }
    if (len) {
      const uint32_t* tw = (const uint32_t*)my_txt;
      uint32_t h = len;
      for (uint32_t i = 0; i < len; i += 4) {
        const uint32_t at = s + i;
        uint32_t d = __builtin_amdgcn_alignbyte(tw[(at >> 2) + 1], tw[at >> 2], at & 3);
        if (len - i < 4) d &= (1u << (8 * (len - i))) - 1u;
        h = long_step(h, d);
      }
      return long_key(p, len, h);
    }
    const uint64_t start = (uint64_t)(p0 + s);
    const uint64_t end = max(doc_limit(start), start);
    len = (uint32_t)(kUtf8 ? long_len_utf8(P.corpus, P.len, start, end) : long_len(P.corpus, P.len, start, end));
    return long_key(p, len, long_hash(p, len));
  };

  // Counts the tokens at [at, at + 64 NX) of the list; nw of them are there.
  auto count = [&](auto nx, uint32_t at, uint32_t nw) -> int {
    constexpr int NX = decltype(nx)::value;
    uint32_t st[NX], wl[NX], e0[NX], e1[NX], one[NX], h[NX];
    bool in[NX];
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
    for (int x = 0; x < NX; ++x) {
      uint64_t lo, hi;
      pack_join(ps[x], lm[x], &lo, &hi);
      key[x] = key4(lo, hi);
      h[x] = red_hash(key[x]);
    }
#pragma unroll
    for (int x = 0; x < NX; ++x)
      if (in[x] && wl[x] - 1 >= 16u) {
        key[x] = long_word(st[x], wl[x]);
        h[x] = place_hash(key[x]);
        wait_vmem();
      }
    return table_add<NX>(T, key, h, one, in);
  };

  while (true) {
    // ---- scan: until the run ends or the table is nearly full ------------------------------
    while (true) {
      if (w0 >= n) {
        // -- the next tile; after it the wave takes whichever no wave has taken
        if (tile_at(kn) >= G1) {
          done = true;
          break;
        }
        p0 = tile_at(kn) - 16;
        uint32_t after = 0;
        if (lane == 0) after = atomicAdd(&s_tile, 1u);
        uint32_t w16;
        const uint4 g = classify16(raw, &w16);
        ((uint4*)my_txt)[lane] = g;
        kn = (uint32_t)__builtin_amdgcn_readfirstlane((int)after);
        raw = load(kn);
        // a bit for each document start in the staged bytes
        uint32_t bnd16 = 0, bnext = 0;
        if (__all(doff < p0)) {
          d0 += 64;
          doff = start_of(d0 + lane);
          if (__all(doff < p0)) seek(p0, d0 + 64);
        }
        const bool here = doff > p0 && doff < p0 + (int64_t)kStripe;
        if (__any(here) || __all(doff < p0 + (int64_t)kStripe)) {
          int64_t o = doff;
          for (uint64_t d = d0;;) {
            if (o > p0 && o < p0 + (int64_t)kStripe)
              atomicOr(&my_bnd[(uint32_t)(o - p0) >> 5], 1u << ((uint32_t)(o - p0) & 31));
            if (!__all(o < p0 + (int64_t)kStripe)) break;
            // (a run of empty documents, which all start here, is passed in a few steps: a million of
            // them in one place, read 64 at a time, took 4.7 ms)
            const int64_t o63 = (int64_t)last_lane64((uint64_t)o);
            d += 64;
            if (__builtin_expect(__all(o == o63), 0)) d = first_from(o63 + 1, d);
            o = start_of(d + lane);
          }
          wave_sync();
          bnd16 = (my_bnd[lane >> 1] >> ((lane & 1) * 16)) & 0xffffu;
          bnext = (my_bnd[(lane + 1) >> 1] >> (((lane + 1) & 1) * 16)) & 0xffffu;  // lane 63: 0
          wave_sync();
          if (lane < kEnds) my_bnd[lane] = 0;
        }
        if (kUtf8 && __any(((g.x | g.y | g.z | g.w) & 0x80808080u) != 0)) {
          const uint32_t next = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)g.x, 0x130, 0xf, 0xf, false);
          const uint32_t res = utf8_mask(g, next, bnd16 | (bnext << 16));
          w16 |= (res & 0xffffu) |
                 (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(res >> 16), 0x138, 0xf, 0xf, false);
        }
        if (p0 < R0 || p0 + (int64_t)kStripe > R1) w16 = cut16(w16, p0 + lane * 16, R0, R1);
        const uint32_t prev = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(w16 >> 15), 0x138, 0xf, 0xf, false);
        // (lane 63: a word that reaches the last byte goes on for all that is known, and is longer
        // than 16 bytes)
        const uint32_t next = (uint32_t)__builtin_amdgcn_update_dpp(1, (int)(w16 & 1u), 0x130, 0xf, 0xf, false);
        start16 = w16 & (~((w16 << 1) | prev) | bnd16) & 0xffffu;
        // the words of other tiles, and of the next workgroup
        if (lane - 1 >= kTile / 16 || p0 + (int64_t)(lane * 16) >= G1) start16 = 0;
        uint32_t last16 = w16 & (~((w16 >> 1) | (next << 15)) | (bnd16 >> 1) | ((bnext & 1u) << 15)) & 0xffffu;
        // (UTF-8: a sequence that runs over the staged text is not known to be one; only words longer
        // than 16 bytes reach the last lane)
        if (kUtf8 && lane == 63) last16 = 0;
        ((uint16_t*)my_ends)[lane] = (uint16_t)last16;
        const uint32_t c = __popc(start16), incl = wave_incl_scan(c);
        rank = incl - c;
        n = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        tokens += n;
        w0 = off = 0;
        continue;
      }
      if (off == 0) {  // list the starts of ranks [w0, w0 + kList)
        list_starts(start16, lane * 16, rank - w0, n <= kList, kList, my_starts);
        wave_sync();
      }
      // a round: two tokens a lane from the list's start, if there are more than 64, one from its
      // 128th (a tile of 176 tokens, usual for English text, took two rounds of 128)
      const uint32_t nw = min(n - w0, kList - off);
      const bool two = off == 0 && nw > 64;
      const int r = two ? count(std::integral_constant<int, 2>(), off, nw)
                        : count(std::integral_constant<int, 1>(), off, nw);
      if (r == kNoRoom && !kSingle) break;  // this round again when the table is empty
      if (r != kAdded) over = true;
      const uint32_t adv = two ? 128 : 64;
      w0 += adv;
      off = off + adv < kList ? off + adv : 0;
      wave_sync();
    }
    if (done && !counted) {
      counted = true;
      if (lane == 0) {
        atomicAdd(&s_done, 1u);
        atomicAdd(&s_tokens, (uint32_t)tokens);
      }
    }
    // ---- the table's words leave -------------------------------------------------------------
    __syncthreads();
    const bool end = s_done == kWaves;
    // (one addition per workgroup: one per wave, 4,096 on one address, took about 40 us)
    if (end && tid == 0) add64(&hdr_of()->total_tokens, s_tokens);
    if (kSingle) {  // (a word that found no room sets kFlagArena below)
      export_table<false>(P, T, true, 1u, s_tmp, &s_base);
      break;
    }
    const uint32_t ne = min(s_nent, T.cap);
    // room for all entries, those without a count too: the answer arrives while they are looked at
    // (lists << 40 | records)
    uint64_t got = 0;
    if (tid == 0) got = atomicAdd((unsigned long long*)&hdr_of()->arena_next, (1ull << 40) | ne);
    uint32_t at[kPerThread];  // partition << 16 | place in it
#pragma unroll
    for (uint32_t x = 0; x < kPerThread; ++x) {
      const uint32_t j = tid + x * kBlk;
      at[x] = kNone;
      if (j < ne && T.cnt[j]) {
        const uint32_t p = part_hash(T.key[j]) & (args()->parts - 1);
        at[x] = (p << 16) | atomicAdd(&s_hist[p], 1u);
      }
    }
    __syncthreads();
    uint32_t cnt = 0, incl = 0;
    if (tid < kParts) {
      cnt = s_hist[tid];
      incl = wave_incl_scan(cnt);
      if (lane == 63) s_scan[wv] = incl;
    }
    __syncthreads();
    if (tid == 0) {
      s_base = got;
      if ((got & ((1ull << 40) - 1)) + ne > args()->cap_recs || (got >> 40) >= args()->max_lists) {
        or32(&hdr_of()->flags, kFlagArena);
        s_base = ~0ull;
      }
    }
    if (tid < kParts) {
      uint32_t b = incl - cnt;
      for (uint32_t w = 0; w < 4; ++w) b += w < wv ? s_scan[w] : 0u;
      s_start[tid] = b;
      s_hist[tid] = 0;
    }
    __syncthreads();
    if (s_base == ~0ull) return;  // the call counts again: nothing more is of use
    const uint64_t list = s_base >> 40;
    const uint32_t rec = (uint32_t)(s_base & ((1ull << 40) - 1));
    if (tid < args()->parts) as_global(args()->dir)[(uint64_t)tid * args()->max_lists + list] = make_uint2(rec + s_start[tid], cnt);
#pragma unroll
    for (uint32_t x = 0; x < kPerThread; ++x) {
      const uint32_t j = tid + x * kBlk;
      if (at[x] == kNone) continue;
      const uint32_t r = rec + s_start[at[x] >> 16] + (at[x] & 0xffffu);
      as_global(args()->rec_key)[r] = T.key[j];
      ((uint32_t*)as_global(args()->rec_cnt))[r] = T.cnt[j];
    }
    __syncthreads();
    if (end) break;
    for (uint32_t j = tid; j < kRedSlots / 4; j += kBlk) ((uint4*)T.slot)[j] = make_uint4(0, 0, 0, 0);
    if (tid == 0) s_nent = 0;
    __syncthreads();
  }
  if (over) or32(&hdr_of()->flags, kFlagArena);
}

// ---------------------------------------------------------------------------------------
// reduce
// ---------------------------------------------------------------------------------------
// One workgroup per partition. The directory rows of kRows lists at a time give the flat order
// of their records; a thread finds its record's list by a binary search in LDS. A partition
// whose words do not fit the LDS table is summed in classes of its hash (two, four, ... classes,
// each reading the records again), so that any number of distinct words is counted in LDS (but for
// long words alike in length and the 24 hash bits of their key, which no split tells apart).
template <class C>
constexpr uint32_t kRedEntries = sizeof(C) == 4 ? kPartRedEntries : kPartMergeEntries;
template <class C>
__global__ __launch_bounds__(kBlk) void part_reduce_kernel(PartParams P) {
  constexpr bool kWide = sizeof(C) == 8;
  constexpr uint32_t kRows = 1024;
  constexpr uint32_t kMaxBits = 16;
  constexpr int kRecs = 2;  // records of a thread read and added together
  extern __shared__ __align__(16) uint8_t s_dyn[];
  __shared__ uint32_t s_pre[kRows + 1], s_rec[kRows];
  __shared__ uint32_t s_nent, s_full;
  __shared__ uint64_t s_tmp[kWaves], s_base;
  Header* const hdr = P.hdr;
  // (flags of the launches before: nothing in this one sets them, so all threads see the same)
  if (ld_relaxed32(&hdr->flags) & (kFlagBadOffsets | kFlagArena)) return;
  PartTable<C> T;
  T.slot = (uint32_t*)s_dyn;
  T.key = (uint4*)(T.slot + kRedSlots);
  T.cnt = (C*)(T.key + kRedEntries<C>);
  T.n = &s_nent;
  T.cap = kRedEntries<C>;
  const uint32_t tid = threadIdx.x;
  const uint32_t lists = (uint32_t)(hdr->arena_next >> 40);
  const uint2* dir = P.dir + (uint64_t)blockIdx.x * P.max_lists;

  // classes of the part hash still to sum: the low `bits` bits above the partition's are `value`
  uint32_t bits = 0, value = 0;
  while (true) {
    for (uint32_t i = tid; i < kRedSlots / 4; i += kBlk) ((uint4*)T.slot)[i] = make_uint4(0, 0, 0, 0);
    if (tid == 0) {
      s_nent = 0;
      s_full = 0;
    }
    for (uint32_t q0 = 0; q0 < lists; q0 += kRows) {
      const uint32_t nq = min(kRows, lists - q0);
      uint2 d = make_uint2(0, 0);
      if (tid < nq) d = dir[q0 + tid];
      uint64_t tot;
      const uint64_t pre = block_scan64(d.y, s_tmp, &tot);  // (its barriers also end the last rows' use)
      s_pre[tid] = (uint32_t)pre;
      s_rec[tid] = d.x;
      if (tid == 0) s_pre[kRows] = (uint32_t)tot;
      __syncthreads();
      const uint32_t m = (uint32_t)tot;
      // A round's records are read while those of the round before are added: two a thread, for the
      // registers (four without reading ahead: reduce of 1 / 20 / 64 MB 12.2 / 17.7 / 69.8 us, of
      // 2,000 tables 23.7; now 10.4 / 16.3 / 58.0, 67.3 before long words were written 16 bytes at a
      // time, and 20.8).
      uint4 k[kRecs], kn[kRecs];
      C c[kRecs], cn[kRecs];
      auto read = [&](uint32_t f0) {
        uint32_t lo[kRecs];
#pragma unroll
        for (int x = 0; x < kRecs; ++x) lo[x] = 0;
#pragma unroll
        for (uint32_t step = kRows / 2; step; step >>= 1)
#pragma unroll
          for (int x = 0; x < kRecs; ++x)  // the last list that starts at or before the record
            if (s_pre[lo[x] + step] <= f0 + x * kBlk + tid) lo[x] += step;
#pragma unroll
        for (int x = 0; x < kRecs; ++x) {
          const uint32_t f = f0 + x * kBlk + tid;
          const uint32_t r = f < m ? s_rec[lo[x]] + (f - s_pre[lo[x]]) : 0u;
          kn[x] = P.rec_key[r];
          cn[x] = ((const C*)P.rec_cnt)[r];
        }
      };
      if (m) read(0);
      for (uint32_t f0 = 0; f0 < m; f0 += kRecs * kBlk) {
        uint32_t h[kRecs];
        bool use[kRecs];
#pragma unroll
        for (int x = 0; x < kRecs; ++x) {
          k[x] = kn[x];
          c[x] = cn[x];
          use[x] = f0 + x * kBlk + tid < m;
        }
        if (f0 + kRecs * kBlk < m) read(f0 + kRecs * kBlk);
#pragma unroll
        for (int x = 0; x < kRecs; ++x) {
          h[x] = place_hash(k[x]);
          if (bits) use[x] &= ((part_hash(k[x]) >> 8) & ((1u << bits) - 1)) == value;
          if (use[x] && is_long_key(k[x])) k[x] = known_key(T, k[x], h[x]);
        }
        if (f0 + (tid & ~63u) < m && table_add<kRecs>(T, k, h, c, use) != kAdded) s_full = 1;
      }
      __syncthreads();
    }
    __syncthreads();
    if (s_full) {
      if (bits == kMaxBits) {
        if (tid == 0) or32(&hdr->flags, kFlagSplit);
        return;
      }
      ++bits;  // this class in two: first the half whose new bit is 0
      __syncthreads();
      continue;
    }
    // the next class: the other half of the smallest split whose first half this one ends
    while (bits && (value >> (bits - 1))) {
      --bits;
      value &= (1u << bits) - 1;
    }
    export_table<kWide>(P, T, bits == 0, gridDim.x, s_tmp, &s_base);
    if (bits == 0) break;
    value |= 1u << (bits - 1);
  }
}

// ---------------------------------------------------------------------------------------
// merge: entries of tables as records
// ---------------------------------------------------------------------------------------
// A workgroup makes one list of kMergeSpan entries of one input: their words are packed, ranked
// inside their partition with one LDS atomic each and written as records (64-bit counts: those of
// the inputs may be wide). Words are not summed here: a (document, word) table holds a word once
// per document, so a few documents' entries hardly repeat.
//
// Adding every entry to one device table instead took 374 us for the tables of 2,000 documents
// (1.4 million entries of 50,000 words): the frequent words are in every document, and their
// slots were hit 2,000 times each. The whole merge of them: 491 -> 86 us (map 30, reduce 29).
__global__ __launch_bounds__(kBlk) void part_merge_kernel(MergeBatch M, PartParams P) {
  constexpr uint32_t kMine = kMergeSpan / kBlk;
  __shared__ uint32_t s_hist[kParts], s_start[kParts], s_scan[4];
  __shared__ uint64_t s_base;
  const uint32_t tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  uint32_t x = 0;
  while (x + 1 < M.n && M.first_block[x + 1] <= blockIdx.x) ++x;
  const MergeInput& in = M.in[x];
  const uint64_t first = (uint64_t)(blockIdx.x - M.first_block[x]) * kMergeSpan;
  if (tid < kParts) s_hist[tid] = 0;
  uint64_t got = 0;
  if (tid == 0) {
    const uint64_t n = min((uint64_t)kMergeSpan, in.n - first);
    got = atomicAdd((unsigned long long*)&P.hdr->arena_next, (1ull << 40) | n);
    s_base = got;
    if ((got & ((1ull << 40) - 1)) + n > P.cap_recs || (got >> 40) >= P.max_lists) {
      or32(&P.hdr->flags, kFlagArena);
      s_base = ~0ull;
    }
  }
  uint4 k[kMine];
  uint64_t c[kMine];
  uint32_t at[kMine];
  const uint8_t* const end = in.words + in.word_offsets[in.n];
#pragma unroll
  for (uint32_t j = 0; j < kMine; ++j) {
    const uint64_t e = first + j * kBlk + tid;
    c[j] = 0;
    k[j] = make_uint4(0, 0, 0, 0);
    if (e < in.n) {
      const uint64_t a = in.word_offsets[e], len = in.word_offsets[e + 1] - a;
      c[j] = in.count_bytes == 4 ? (uint64_t)(int64_t)((const int32_t*)in.counts)[e]
                                 : (uint64_t)((const int64_t*)in.counts)[e];
      const uint8_t* w = in.words + a;
      if (len == 0) {
        c[j] = 0;
      } else {
        uint64_t lo = 0, hi = 0xffull << 56;
        if (len <= 16) load_packed(w, (uint32_t)len, end, &lo, &hi);
        k[j] = key4(lo, hi);
        if (is_long_key(k[j])) k[j] = long_key(w, (uint32_t)len, long_hash(w, (uint32_t)len));
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (uint32_t j = 0; j < kMine; ++j) {
    at[j] = kNone;
    if (c[j]) {
      const uint32_t p = part_hash(k[j]) & (P.parts - 1);
      at[j] = (p << 16) | atomicAdd(&s_hist[p], 1u);
    }
  }
  __syncthreads();
  uint32_t cnt = 0, incl = 0;
  if (tid < kParts) {
    cnt = s_hist[tid];
    incl = wave_incl_scan(cnt);
    if (lane == 63) s_scan[wv] = incl;
  }
  __syncthreads();
  if (tid < kParts) {
    uint32_t b = incl - cnt;
    for (uint32_t w = 0; w < 4; ++w) b += w < wv ? s_scan[w] : 0u;
    s_start[tid] = b;
  }
  __syncthreads();
  if (s_base == ~0ull) return;
  const uint64_t list = s_base >> 40;
  const uint32_t rec = (uint32_t)(s_base & ((1ull << 40) - 1));
  if (tid < P.parts) P.dir[(uint64_t)tid * P.max_lists + list] = make_uint2(rec + s_start[tid], cnt);
#pragma unroll
  for (uint32_t j = 0; j < kMine; ++j) {
    if (at[j] == kNone) continue;
    const uint32_t r = rec + s_start[at[j] >> 16] + (at[j] & 0xffffu);
    P.rec_key[r] = k[j];
    ((uint64_t*)P.rec_cnt)[r] = c[j];
  }
}

size_t part_map_dyn() { return (size_t)kRedSlots * 4 + (size_t)kPartMapEntries * 20 + kWaves * kText; }
template <class C>
size_t part_reduce_dyn() { return (size_t)kRedSlots * 4 + (size_t)kRedEntries<C> * (16 + sizeof(C)); }

hipError_t set_part_smem() {
  static const hipError_t once = [] {
    const struct { const void* f; size_t dyn; } k[6] = {
        {(const void*)part_map_kernel<false, false>, part_map_dyn()},
        {(const void*)part_map_kernel<true, false>, part_map_dyn()},
        {(const void*)part_map_kernel<false, true>, part_map_dyn()},
        {(const void*)part_map_kernel<true, true>, part_map_dyn()},
        {(const void*)part_reduce_kernel<uint32_t>, part_reduce_dyn<uint32_t>()},
        {(const void*)part_reduce_kernel<uint64_t>, part_reduce_dyn<uint64_t>()}};
    hipError_t e = hipSuccess;
    for (int i = 0; i < 6 && e == hipSuccess; ++i)
      e = hipFuncSetAttribute(k[i].f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)k[i].dyn);
    return e;
  }();
  return once;
}

template <bool kSingle>
static hipError_t launch_map(const PartParams& P, uint32_t grid, hipStream_t s) {
  if (P.utf8)
    hipLaunchKernelGGL((part_map_kernel<kSingle, true>), dim3(grid), dim3(kBlk), part_map_dyn(), s, P);
  else
    hipLaunchKernelGGL((part_map_kernel<kSingle, false>), dim3(grid), dim3(kBlk), part_map_dyn(), s, P);
  return hipGetLastError();
}
hipError_t launch_part_map(const PartParams& P, uint32_t grid, hipStream_t s) {
  return launch_map<false>(P, grid, s);
}
hipError_t launch_part_single(const PartParams& P, hipStream_t s) { return launch_map<true>(P, 1, s); }
hipError_t launch_part_reduce(const PartParams& P, hipStream_t s) {
  hipLaunchKernelGGL(part_reduce_kernel<uint32_t>, dim3(P.parts), dim3(kBlk),
                     part_reduce_dyn<uint32_t>(), s, P);
  return hipGetLastError();
}

hipError_t launch_part_merge(const MergeInput* in, uint32_t k, const PartParams& P, hipStream_t s) {
  hipError_t e = set_part_smem();
  if (e != hipSuccess) return e;
  e = for_merge_batches(in, k, kMergeSpan, [&](const MergeBatch& M, uint32_t blocks) {
    hipLaunchKernelGGL(part_merge_kernel, dim3(blocks), dim3(kBlk), 0, s, M, P);
    return hipGetLastError();
  });
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(part_reduce_kernel<uint64_t>, dim3(P.parts), dim3(kBlk),
                     part_reduce_dyn<uint64_t>(), s, P);
  return hipGetLastError();
}

}  // namespace wc
