// Words as 16-byte keys, long ones included, and the LDS table that counts them, shared by the
// partitioned count and the per-document count.
#pragma once

#include "wc_internal.h"
#include "wc_stripe.h"
#include "wc_utf8.h"

namespace wc {

constexpr uint32_t kNone = 0xffffffffu;

// A word of at most 16 bytes is its packed bytes; a longer one the address of an occurrence, its
// length (below 2^32) and 24 bits of its hash under a top byte of 0xff, which no word byte of
// either tokeniser is. (With the hash in the key a long word is read again only to be compared
// with one of the same length and hash.) An address has 48 bits; the 16 above them are the
// caller's and part of the key.
WC_DEV uint4 long_key(const uint8_t* p, uint32_t n, uint32_t h) {
  return key4((uint64_t)(uintptr_t)p, n | ((uint64_t)((h ^ (h >> 24)) & 0xffffffu) << 32) | (0xffull << 56));
}
WC_DEV bool is_long_key(const uint4 k) { return (k.w >> 24) == 0xffu; }
WC_DEV const uint8_t* long_ptr(const uint4 k) {
  return as_global_lane((const uint8_t*)(uintptr_t)((uint64_t)k.x | ((uint64_t)(k.y & 0xffffu) << 32)));
}

WC_DEV uint32_t mix32(uint32_t h) {  // the 32-bit finaliser of MurmurHash3 (Appleby)
  h ^= h >> 16;
  h *= 0x85EBCA6Bu;
  h ^= h >> 13;
  h *= 0xC2B2AE35u;
  h ^= h >> 16;
  return h;
}
// Two hashes of a key: one for its place in the LDS tables, one for its partition (the low 8
// bits) and, above those, for splitting a partition that does not fit LDS.
WC_DEV uint32_t place_hash(const uint4 k) {
  const uint4 l = make_uint4(k.z, k.w, k.y >> 16, 0u);
  return red_hash(is_long_key(k) ? l : k);
}
WC_DEV uint32_t part_hash(const uint4 k) {
  const uint32_t s = (k.x ^ __builtin_amdgcn_alignbit(k.y, k.y, 21)) +
                     (k.z ^ __builtin_amdgcn_alignbit(k.w, k.w, 13));
  return mix32(is_long_key(k) ? k.z ^ __builtin_amdgcn_alignbit(k.w, k.w, 13) : s);
}

// Hash of a long word: its folded bytes four at a time, the last ones zero padded.
WC_DEV uint32_t long_step(uint32_t h, uint32_t d) {
  h = (h ^ d) * 0x9E3779B1u;
  return h ^ (h >> 15);
}
// the same of a word in device memory
WC_DEV uint32_t long_hash(const uint8_t* p, uint32_t n) {
  uint32_t h = n, i = 0, f;
  for (; i + 16 <= n; i += 16) {
    uint32_t d[4];
    __builtin_memcpy(d, p + i, 16);
#pragma unroll
    for (int j = 0; j < 4; ++j) h = long_step(h, fold_classify4(d[j], &f));
  }
  for (; i < n; i += 4) {
    uint32_t d = 0;
    for (uint32_t q = 0; q < 4 && i + q < n; ++q) d |= (uint32_t)p[i + q] << (8 * q);
    h = long_step(h, fold_classify4(d, &f));
  }
  return h;
}
// Length of the word at position s that ends at `end` (its document's end) at the latest.
WC_DEV uint64_t long_len(const uint8_t* corpus, uint64_t len, uint64_t s, uint64_t end) {
  uint64_t p = s;
  while (p < end) {
    // up to 64 bytes at once, from the 16-byte block holding p on
    const int64_t a = (int64_t)p - (int64_t)((uintptr_t)(corpus + p) & 15);
    uint32_t m[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) classify16(load_text16(corpus, len, a + 16 * j), &m[j]);
    uint64_t w = (uint64_t)(m[0] | (m[1] << 16)) | ((uint64_t)(m[2] | (m[3] << 16)) << 32);
    const uint32_t k = (uint32_t)((int64_t)p - a);
    w = ~w >> k;  // first delimiter from p on
    if (w) return min(p + (uint64_t)__ffsll((unsigned long long)w) - 1, end) - s;
    p += 64 - k;
  }
  return end - s;
}

// Two words of n > 16 bytes: compared 32 bytes at a time, from both ends of what is left so that
// nothing past a word is read and all loads of a step are in flight together.
WC_DEV bool long_same(const uint8_t* a, const uint8_t* b, uint32_t n) {
  if (a == b) return true;
  while (true) {
    uint32_t x[8], y[8], f, d = 0;
    const uint32_t tail = n < 32 ? n - 16 : 16;
    __builtin_memcpy(x, a, 16);
    __builtin_memcpy(y, b, 16);
    __builtin_memcpy(x + 4, a + tail, 16);
    __builtin_memcpy(y + 4, b + tail, 16);
#pragma unroll
    for (int j = 0; j < 8; ++j) d |= fold_classify4(x[j], &f) ^ fold_classify4(y[j], &f);
    if (d) return false;
    if (n <= 32) return true;
    const uint32_t step = min(32u, n - 16);  // (the next 16 bytes at least are the word's)
    a += step;
    b += step;
    n -= step;
  }
}
// The same under the UTF-8 reading.
WC_DEV uint64_t long_len_utf8(const uint8_t* corpus, uint64_t len, uint64_t s, uint64_t end) {
  uint64_t p = s;
  uint32_t over = 0;  // bytes of the next block that end a sequence of this one
  while (p < end) {
    const int64_t a = (int64_t)p - (int64_t)((uintptr_t)(corpus + p) & 15);
    uint32_t m;
    const uint4 g = classify16(load_text16(corpus, len, a), &m);
    const uint32_t next = load_text4(corpus, len, a + 16);
    const int64_t left = (int64_t)end - a;
    const uint32_t stop = left < 19 ? 1u << left : 0u;  // the document's end
    const uint32_t res = utf8_mask(g, next, stop);
    m |= (res & 0xffffu) | over;
    over = res >> 16;
    const uint32_t k = (uint32_t)((int64_t)p - a);
    const uint32_t w = (~m & 0xffffu) >> k;
    if (w) return min(p + (uint64_t)__ffs(w) - 1, end) - s;
    p += 16 - k;
  }
  return end - s;
}

WC_DEV bool same_key(const uint4 a, const uint4 b) {
  if (key_eq(a, b)) return true;
  return is_long_key(a) && a.z == b.z && a.w == b.w && (a.y >> 16) == (b.y >> 16) &&
         long_same(long_ptr(a), long_ptr(b), a.z);
}

// ---- the LDS table -----------------------------------------------------------------------
template <class Count, uint32_t kTableSlots = kRedSlots>
struct PartTable {
  using C = Count;
  static constexpr uint32_t kSlots = kTableSlots, kGroups = kSlots / 4;
  // the home group of a hash: its top bits
  static WC_DEV uint32_t group(uint32_t h) { return h >> (32 - __builtin_ctz(kGroups)); }
  uint32_t* slot;  // [kSlots], 0 = empty
  uint4* key;      // [cap]
  C* cnt;          // [cap]
  uint32_t* n;     // entries handed out (may pass cap)
  uint32_t cap;
};
WC_DEV void lds_add(uint32_t* p, uint32_t v) { atomicAdd(p, v); }
WC_DEV void lds_add(uint64_t* p, uint64_t v) {
  atomicAdd((unsigned long long*)p, (unsigned long long)v);
}

// The tag-slot table of wc_stripe.h (counts of type C). An entry's key and count are written before its slot is
// claimed (a wave's LDS accesses are in order), so a claimed slot shows its key and entries need
// no clearing; an entry whose key turned out to have another keeps count 0.

// A key that table_add could not place in its first two groups, with an entry already taken for
// it. Every iteration finds the key, claims a slot, loses a slot of the group to another key (at
// most four times) or moves to the next group. (At 5,120 entries in 8,192 slots a run of 16 full
// groups is met about once in a million groups, which is several times in a text of 64 MB.)
template <class Table>
WC_DEV bool part_add(const Table& T, const uint4 want, uint32_t h, typename Table::C n, uint32_t mine) {
  constexpr uint32_t kGroups = Table::kGroups;
  const uint32_t tag = red_tag(h);
  uint32_t g = Table::group(h), probe = 0;
  bool active = true, ok = false;
  while (__any(active)) {
    bool claim = false;
    int free_j = -1;
    if (active) {
      const uint4 s4 = ((const uint4*)T.slot)[g];
      const uint32_t e[4] = {s4.x, s4.y, s4.z, s4.w};
      bool found = false;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (found) continue;
        if ((e[j] >> 13) == tag) {
          const uint32_t idx = e[j] & 0x1fffu;
          if (same_key(T.key[idx], want)) {
            lds_add(&T.cnt[idx], n);
            found = true;
          }
        } else if (e[j] == 0 && free_j < 0) {
          free_j = j;
        }
      }
      if (found) {
        T.cnt[mine] = 0;
        ok = true;
        active = false;
      } else if (free_j >= 0) {
        claim = true;
      } else {
        g = (g + 1) & (kGroups - 1);
        if (++probe >= kGroups) active = false;  // (never: there are more slots than entries)
      }
    }
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    if (claim && atomicCAS(&T.slot[g * 4 + free_j], 0u, (tag << 13) | mine) == 0) {
      ok = true;
      active = false;
    }
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
  }
  if (!ok) T.cnt[mine] = 0;
  return ok;
}

WC_DEV uint32_t pick4(const uint4 g, uint32_t tag) {  // the first slot with the tag, or 0
  uint32_t m = 0u;
  m = (g.w >> 13) == tag ? g.w : m;
  m = (g.z >> 13) == tag ? g.z : m;
  m = (g.y >> 13) == tag ? g.y : m;
  m = (g.x >> 13) == tag ? g.x : m;
  return m;
}

// Entry of a key, or -1 (claimed slots of a group are a prefix). While others add to the table, a key
// that they have only just added may not be found.
template <class Table>
WC_DEV int table_find(const Table& T, const uint4 want, uint32_t h) {
  constexpr uint32_t kGroups = Table::kGroups;
  const uint32_t tag = red_tag(h);
  uint32_t g = Table::group(h);
  for (uint32_t probe = 0; probe < kGroups; ++probe) {
    const uint4 s4 = ((const uint4*)T.slot)[g];
    const uint32_t e[4] = {s4.x, s4.y, s4.z, s4.w};
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if ((e[j] >> 13) == tag && same_key(T.key[e[j] & 0x1fffu], want)) return (int)(e[j] & 0x1fffu);
    if (s4.w == 0) return -1;
    g = (g + 1) & (kGroups - 1);
  }
  return -1;
}

// The key of a word of more than 16 bytes, as the table has it if it does: under the address of the
// occurrence that took the entry. table_add compares keys, and a word under another address takes
// an entry that part_add, which finds the word by its content, leaves unused. For the reduce,
// where a table may get a word thousands of times (once per list; per document in a merge) and
// has nowhere to put what does not fit. (A test of every key inside table_add cost 1.5 to 3.5 % of
// a count; in the scans, whose tables may fill up, the second search cost 0.4 to 1 %.)
template <class Table>
WC_DEV uint4 known_key(const Table& T, const uint4 key, uint32_t h) {
  const int i = table_find(T, key, h);
  return i >= 0 ? T.key[i] : key;
}

// Adds n[x] occurrences of key[x] (hash h[x]) for the lanes and x with f[x]; called by whole
// waves. kNoRoom: the entries ran out, and nothing was counted, or, with kPartial, the keys
// that have an entry were and `left` says which were not; kNoSlot: some key found no slot.
//
// Each LDS step is taken for all N keys of a lane before any is waited for: the home group, the
// key of its first tag match, and, for the lanes whose home group is full without the key, the
// same of the next group. Then the new keys of the whole wave take entries with one atomic and
// claim slots from the first free one of their group on, where a lost claim's answer is the
// slot's occupant: compared when its tag matches, passed by otherwise, without reading the
// group again. (Before, each key of the lanes went through an entry, a claim and, for what was
// left, the loop of part_add by itself: map of a 20 MB text 62 -> 55 us, of a 64 MB text 271 -> 181.)
//
// spare[N], when given, starts as kNone with an empty table: an entry taken for a word that another
// lane has claimed is kept for the lane's next new word. (The first words of a table, new to all
// waves at once, take many: without it the per-document kernel's groups of 48 KiB spilled more
// often, 5.87 -> 5.46 ms for 100,000 documents, and some of 34 KiB did, 107 -> 74 us for 2,000.)
constexpr int kAdded = 0, kNoRoom = 1, kNoSlot = 2;
template <int N, bool kPartial = false, class Table>
WC_DEV int table_add(const Table& T, const uint4 (&key)[N], const uint32_t (&h)[N],
                     const typename Table::C (&n)[N], const bool (&f)[N], bool* left = nullptr,
                     uint32_t* spare = nullptr) {
  using C = typename Table::C;
  constexpr uint32_t kGroups = Table::kGroups;
  const uint32_t lane = threadIdx.x & 63;
  uint4 g[N], k[N];
  uint32_t e[N], gi[N], tag[N];
  bool hit[N], next[N];
#pragma unroll
  for (int x = 0; x < N; ++x) {
    gi[x] = Table::group(h[x]);
    g[x] = ((const uint4*)T.slot)[gi[x]];
  }
#pragma unroll
  for (int x = 0; x < N; ++x) pin(g[x]);
#pragma unroll
  for (int x = 0; x < N; ++x) {
    tag[x] = red_tag(h[x]);
    e[x] = pick4(g[x], tag[x]);
    k[x] = T.key[e[x] & 0x1fffu];
  }
#pragma unroll
  for (int x = 0; x < N; ++x) pin(k[x]);
  bool more = false;
#pragma unroll
  for (int x = 0; x < N; ++x) {
    const bool eq = key_eq(k[x], key[x]);
    hit[x] = f[x] & (e[x] != 0) & eq;
    next[x] = f[x] & (e[x] == 0) & (g[x].w != 0);  // (claimed slots of a group are a prefix)
    more |= next[x];
  }
  if (__any(more)) {
#pragma unroll
    for (int x = 0; x < N; ++x) {
      if (next[x]) {
        gi[x] = (gi[x] + 1) & (kGroups - 1);
        g[x] = ((const uint4*)T.slot)[gi[x]];
        e[x] = pick4(g[x], tag[x]);
        if (e[x] != 0) hit[x] = key_eq(T.key[e[x] & 0x1fffu], key[x]);
      }
    }
  }
  uint64_t mm[N];
  uint32_t tot = 0;
  bool miss[N], some = false;
#pragma unroll
  for (int x = 0; x < N; ++x) {
    miss[x] = f[x] && !hit[x];
    some |= miss[x];
    mm[x] = __ballot(miss[x] && (!spare || spare[x] == kNone));
    tot += (uint32_t)__popcll(mm[x]);
  }
  uint32_t base = 0;
  if (tot) {
    if (lane == 0) base = atomicAdd(T.n, tot);
    base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
    if (base + tot > T.cap) {
      // the entries taken stay unused (giving them back could take a later wave's from the end)
      for (uint32_t i = base + lane; i < min(base + tot, T.cap); i += 64) T.cnt[i] = 0;
      if (kPartial) {
#pragma unroll
        for (int x = 0; x < N; ++x) {
          if (hit[x]) lds_add(&T.cnt[e[x] & 0x1fffu], n[x]);
          left[x] = miss[x];
        }
      }
      return kNoRoom;
    }
  }
#pragma unroll
  for (int x = 0; x < N; ++x)
    if (hit[x]) lds_add(&T.cnt[e[x] & 0x1fffu], n[x]);
  if (!__any(some)) return kAdded;
  uint32_t mine[N], at[N];
  bool act[N], any = false, slow = false;
#pragma unroll
  for (int x = 0; x < N; ++x) {
    mine[x] = base + __builtin_amdgcn_mbcnt_hi((uint32_t)(mm[x] >> 32),
                                               __builtin_amdgcn_mbcnt_lo((uint32_t)mm[x], 0u));
    base += (uint32_t)__popcll(mm[x]);
    if (spare && miss[x]) {
      if (spare[x] != kNone) mine[x] = spare[x];
      spare[x] = kNone;
    }
    const uint32_t used = (g[x].x != 0) + (g[x].y != 0) + (g[x].z != 0) + (g[x].w != 0);
    at[x] = gi[x] * 4 + used;
    if (miss[x]) {
      T.key[mine[x]] = key[x];
      T.cnt[mine[x]] = n[x];
    }
    act[x] = miss[x] & (e[x] == 0) & (used < 4);
    any |= act[x];
  }
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  while (__any(any)) {
    uint32_t prev[N];
    bool lost = false;
#pragma unroll
    for (int x = 0; x < N; ++x) {
      prev[x] = 0;
      if (act[x]) prev[x] = atomicCAS(&T.slot[at[x]], 0u, (tag[x] << 13) | mine[x]);
    }
#pragma unroll
    for (int x = 0; x < N; ++x) {
      miss[x] &= !(act[x] & (prev[x] == 0));
      act[x] &= prev[x] != 0;
      lost |= act[x];
    }
    if (!__any(lost)) break;
    // most often the same new word in another lane
    uint4 k2[N];
#pragma unroll
    for (int x = 0; x < N; ++x) k2[x] = T.key[prev[x] & 0x1fffu];
#pragma unroll
    for (int x = 0; x < N; ++x) pin(k2[x]);
    any = false;
#pragma unroll
    for (int x = 0; x < N; ++x) {
      const bool same = act[x] & ((prev[x] >> 13) == tag[x]);
      const bool eq = same & key_eq(k2[x], key[x]);
      if (eq) {
        lds_add(&T.cnt[prev[x] & 0x1fffu], n[x]);
        T.cnt[mine[x]] = 0;
        if (spare) spare[x] = mine[x];
      }
      miss[x] &= !eq;
      at[x] += act[x] ? 1 : 0;
      act[x] = act[x] & !same & ((at[x] & 3u) != 0);
      any |= act[x];
    }
  }
#pragma unroll
  for (int x = 0; x < N; ++x) slow |= miss[x];
  bool ok = true;
  if (__any(slow)) {
    // (one copy of the loop: the values of the next x move to the first's place)
    uint4 kk[N];
    uint32_t hh[N], mi[N];
    C nn[N];
    bool ss[N];
#pragma unroll
    for (int x = 0; x < N; ++x) {
      kk[x] = key[x];
      hh[x] = h[x];
      nn[x] = n[x];
      mi[x] = mine[x];
      ss[x] = miss[x];
    }
#pragma unroll 1
    for (int x = 0; x < N; ++x) {
      if (ss[0]) ok &= part_add(T, kk[0], hh[0], nn[0], mi[0]);
#pragma unroll
      for (int y = 0; y + 1 < N; ++y) {
        kk[y] = kk[y + 1];
        hh[y] = hh[y + 1];
        nn[y] = nn[y + 1];
        mi[y] = mi[y + 1];
        ss[y] = ss[y + 1];
      }
    }
  }
  return __all(ok) ? kAdded : kNoSlot;
}

// The bytes of a packed word of 1..16 bytes to any address: at most two stores of each width, the
// second overlapping the first.
WC_DEV void store_word(uint8_t* dst, uint64_t lo, uint64_t hi, uint32_t n) {
  if (n >= 8) {
    __builtin_memcpy(dst, &lo, 8);
    const uint32_t s = 8 * (n - 8);
    const uint64_t v = s == 0 ? lo : s == 64 ? hi : (lo >> s) | (hi << (64 - s));
    __builtin_memcpy(dst + n - 8, &v, 8);
  } else if (n >= 4) {
    const uint32_t a = (uint32_t)lo, b = (uint32_t)(lo >> (8 * (n - 4)));
    __builtin_memcpy(dst, &a, 4);
    __builtin_memcpy(dst + n - 4, &b, 4);
  } else {
    if (n >= 2) {
      const uint16_t a = (uint16_t)lo;
      __builtin_memcpy(dst, &a, 2);
    }
    if (n != 2) dst[n - 1] = (uint8_t)(lo >> (8 * (n - 1)));
  }
}

// The folded bytes of a word of n >= 16 bytes, 16 at a time, the last 16 overlapping those before.
// (Byte by byte, a read at a time in flight, a partition's 2,900 words of 38 bytes took 100 us.)
WC_DEV void store_long(uint8_t* dst, const uint8_t* src, uint64_t n) {
  for (uint64_t i = 0;;) {
    uint32_t d[4], f;
    __builtin_memcpy(d, src + i, 16);
#pragma unroll
    for (int j = 0; j < 4; ++j) d[j] = fold_classify4(d[j], &f);
    __builtin_memcpy(dst + i, d, 16);
    if (i + 16 == n) return;
    i = min(i + 16, n - 16);
  }
}

WC_DEV uint64_t key_len(const uint4 k) {
  if (is_long_key(k)) return k.z;
  return packed_len((uint64_t)k.x | ((uint64_t)k.y << 32), (uint64_t)k.z | ((uint64_t)k.w << 32));
}


}  // namespace wc
