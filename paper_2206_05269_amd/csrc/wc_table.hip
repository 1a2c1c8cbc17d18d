// Table kernels: compaction of a hash table into dense arrays, per-document CSR grouping,
// merging word tables (Section 3.3: grouped counts of one word are summed), the per-corpus
// distinctive-word ranking (Section 4.3) and the FNV-1a 64 check entry point.

#include "wc_internal.h"

namespace wc {

// ------------------------------------------------------------------------------------------
// fill
// ------------------------------------------------------------------------------------------
__global__ void fill_zero_kernel(uint4* p, uint64_t n16, uint8_t* tail, uint32_t n_tail) {
  uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x;
  uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (; i < n16; i += stride) p[i] = make_uint4(0, 0, 0, 0);
  if (blockIdx.x == 0 && threadIdx.x < n_tail) tail[threadIdx.x] = 0;
}

hipError_t launch_fill_zero(void* p, uint64_t bytes, hipStream_t s) {
  if (bytes == 0) return hipSuccess;
  // p is 16-byte aligned by construction (workspace regions are 256-byte aligned)
  uint64_t n16 = bytes / 16;
  uint32_t n_tail = (uint32_t)(bytes % 16);
  uint64_t blocks = (n16 + 255) / 256;
  if (blocks > 8192) blocks = 8192;
  if (blocks == 0) blocks = 1;
  hipLaunchKernelGGL(fill_zero_kernel, dim3((uint32_t)blocks), dim3(256), 0, s, (uint4*)p, n16,
                     (uint8_t*)p + n16 * 16, n_tail);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// export
// ------------------------------------------------------------------------------------------
WC_DEV uint64_t slot_len(const Slot& sl) {
  if (sl.w0 & kTop) return sl.w1 & ~kTop;
  return packed_len(sl.w0, sl.w1 & ~kTop);
}

template <int BLOCK>
WC_DEV uint64_t block_excl_scan(uint64_t v, uint64_t* s_tmp, uint64_t* total) {
  // s_tmp: BLOCK/64 entries
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint64_t incl = v;
  for (int d = 1; d < 64; d <<= 1) {
    uint64_t y = __shfl_up(incl, d, 64);
    if (lane >= d) incl += y;
  }
  if (lane == 63) s_tmp[wave] = incl;
  __syncthreads();
  uint64_t base = 0, tot = 0;
  for (int w = 0; w < BLOCK / 64; ++w) {
    uint64_t x = s_tmp[w];
    base += w < wave ? x : 0;
    tot += x;
  }
  __syncthreads();
  *total = tot;
  return base + incl - v;
}

__global__ __launch_bounds__(kExportBlock) void export_count_kernel(ExportParams E) {
  __shared__ uint64_t s_a[kExportBlock / 64], s_b[kExportBlock / 64];
  const uint64_t b = blockIdx.x;
  // only the block's totals are needed here, so slots are read wave-contiguously (consecutive
  // lanes, consecutive slots) rather than in the write kernel's per-thread runs
  const uint64_t first = b * kExportSpan + threadIdx.x;
  uint64_t n = 0, bytes = 0;
  for (uint32_t j = 0; j < kExportItems; ++j) {
    uint64_t i = first + (uint64_t)j * kExportBlock;
    if (i < E.slots) {
      Slot sl = E.table[i];
      if (sl.key) {
        ++n;
        bytes += slot_len(sl);
      }
    }
  }
  uint64_t tn, tb;
  block_excl_scan<kExportBlock>(n, s_a, &tn);
  block_excl_scan<kExportBlock>(bytes, s_b, &tb);
  if (threadIdx.x == 0) {
    E.block_sums[2 * b] = tn;
    E.block_sums[2 * b + 1] = tb;
  }
}

__global__ __launch_bounds__(1024) void export_scan_kernel(ExportParams E) {
  __shared__ uint64_t s_a[16], s_b[16];
  __shared__ uint64_t s_carry[2];
  if (threadIdx.x == 0) s_carry[0] = s_carry[1] = 0;
  __syncthreads();
  for (uint64_t base = 0; base < E.n_blocks; base += 1024) {
    uint64_t i = base + threadIdx.x;
    uint64_t a = i < E.n_blocks ? E.block_sums[2 * i] : 0;
    uint64_t b = i < E.n_blocks ? E.block_sums[2 * i + 1] : 0;
    uint64_t ta, tb;
    uint64_t ea = block_excl_scan<1024>(a, s_a, &ta);
    uint64_t eb = block_excl_scan<1024>(b, s_b, &tb);
    if (i < E.n_blocks) {
      E.block_sums[2 * i] = ea + s_carry[0];
      E.block_sums[2 * i + 1] = eb + s_carry[1];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      s_carry[0] += ta;
      s_carry[1] += tb;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    E.hdr->n_entries = s_carry[0];
    E.hdr->word_bytes = s_carry[1];
    if (E.word_offsets) E.word_offsets[s_carry[0]] = s_carry[1];
    if (s_carry[1] > E.word_cap) E.hdr->flags |= kFlagWordCap;
  }
}

__global__ __launch_bounds__(kExportBlock) void export_write_kernel(ExportParams E) {
  __shared__ uint64_t s_a[kExportBlock / 64], s_b[kExportBlock / 64];
  const uint64_t b = blockIdx.x;
  const uint64_t first = b * kExportSpan + (uint64_t)threadIdx.x * kExportItems;
  Slot sl[kExportItems];
  uint64_t n = 0, bytes = 0;
  for (uint32_t j = 0; j < kExportItems; ++j) {
    uint64_t i = first + j;
    sl[j].key = 0;
    if (i < E.slots) {
      sl[j] = E.table[i];
      if (sl[j].key) {
        ++n;
        bytes += slot_len(sl[j]);
      }
    }
  }
  uint64_t tn, tb;
  uint64_t e = block_excl_scan<kExportBlock>(n, s_a, &tn) + E.block_sums[2 * b];
  uint64_t pos = block_excl_scan<kExportBlock>(bytes, s_b, &tb) + E.block_sums[2 * b + 1];
  const bool write_words = (E.hdr->flags & kFlagWordCap) == 0;
  for (uint32_t j = 0; j < kExportItems; ++j) {
    if (!sl[j].key) continue;
    const uint64_t i = first + j;
    uint64_t len = slot_len(sl[j]);
    uint64_t c = (E.per_doc ? (sl[j].cnt & 0xffffffffull) : sl[j].cnt) + E.count_bias;
    E.word_offsets[e] = pos;
    if (E.count_bytes == 4) {
      if (c > 0x7fffffffull) or32(&E.hdr->flags, kFlagCountOverflow);
      ((int32_t*)E.counts)[e] = (int32_t)c;
    } else {
      ((int64_t*)E.counts)[e] = (int64_t)c;
    }
    if (E.per_doc) E.docs[e] = (sl[j].cnt >> 32) - 1;
    if (E.slot_of_entry) E.slot_of_entry[e] = i;
    if (E.entry_of_slot) E.entry_of_slot[i] = e;
    if (write_words) {
      if (sl[j].w0 & kTop) {
        const uint8_t* src = (const uint8_t*)(uintptr_t)(sl[j].w0 & ~kTop);
        for (uint64_t q = 0; q < len; ++q) E.words[pos + q] = (uint8_t)fold_byte(src[q]);
      } else {
        uint64_t lo = sl[j].w0, hi = sl[j].w1 & ~kTop;
        for (uint64_t q = 0; q < len; ++q)
          E.words[pos + q] = (uint8_t)((q < 8 ? lo >> (8 * q) : hi >> (8 * (q - 8))) & 0xff);
      }
    }
    ++e;
    pos += len;
  }
}

// Dense list of the occupied slots with their documents (per-document export, first step).
__global__ __launch_bounds__(kExportBlock) void export_list_kernel(ExportParams E) {
  __shared__ uint64_t s_a[kExportBlock / 64];
  const uint64_t b = blockIdx.x;
  const uint64_t first = b * kExportSpan + (uint64_t)threadIdx.x * kExportItems;
  uint64_t keys[kExportItems], cnts[kExportItems];
  uint64_t n = 0;
  for (uint32_t j = 0; j < kExportItems; ++j) {
    uint64_t i = first + j;
    keys[j] = 0;
    if (i < E.slots) {
      keys[j] = E.table[i].key;
      cnts[j] = E.table[i].cnt;
      n += keys[j] != 0;
    }
  }
  uint64_t tn;
  uint64_t e = block_excl_scan<kExportBlock>(n, s_a, &tn) + E.block_sums[2 * b];
  for (uint32_t j = 0; j < kExportItems; ++j) {
    if (!keys[j]) continue;
    E.docs[e] = (cnts[j] >> 32) - 1;
    E.slot_of_entry[e] = first + j;
    ++e;
  }
}

hipError_t launch_export_list(const ExportParams& E, hipStream_t s) {
  uint32_t nb = (uint32_t)E.n_blocks;
  hipLaunchKernelGGL(export_count_kernel, dim3(nb), dim3(kExportBlock), 0, s, E);
  hipLaunchKernelGGL(export_scan_kernel, dim3(1), dim3(1024), 0, s, E);
  hipLaunchKernelGGL(export_list_kernel, dim3(nb), dim3(kExportBlock), 0, s, E);
  return hipGetLastError();
}

// Lengths of the words of slots listed in entry order (lens[n] = 0 closes the scan).
__global__ void slot_lens_kernel(const Slot* table, const uint64_t* slots, uint64_t n,
                                 uint64_t* lens) {
  uint64_t e = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x;
  if (e > n) return;
  lens[e] = e < n ? slot_len(table[slots[e]]) : 0;
}

// Write entry e from slot slots[e]: count, document, word bytes at word_offsets[e].
__global__ void slot_write_kernel(const Slot* table, const uint64_t* slots, uint64_t n,
                                  const uint64_t* word_offsets, uint8_t* words, void* counts,
                                  uint32_t count_bytes, uint64_t count_bias, uint64_t* docs,
                                  Header* hdr) {
  uint64_t e = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x;
  if (e >= n) return;
  Slot sl = table[slots[e]];
  uint64_t c = (sl.cnt & 0xffffffffull) + count_bias;
  if (count_bytes == 4) {
    if (c > 0x7fffffffull) or32(&hdr->flags, kFlagCountOverflow);
    ((int32_t*)counts)[e] = (int32_t)c;
  } else {
    ((int64_t*)counts)[e] = (int64_t)c;
  }
  docs[e] = (sl.cnt >> 32) - 1;
  uint64_t pos = word_offsets[e], len = word_offsets[e + 1] - pos;
  if (sl.w0 & kTop) {
    const uint8_t* src = (const uint8_t*)(uintptr_t)(sl.w0 & ~kTop);
    for (uint64_t q = 0; q < len; ++q) words[pos + q] = (uint8_t)fold_byte(src[q]);
  } else {
    uint64_t lo = sl.w0, hi = sl.w1 & ~kTop;
    for (uint64_t q = 0; q < len; ++q)
      words[pos + q] = (uint8_t)((q < 8 ? lo >> (8 * q) : hi >> (8 * (q - 8))) & 0xff);
  }
}

hipError_t launch_slot_lens(const Slot* table, const uint64_t* slots, uint64_t n, uint64_t* lens,
                            hipStream_t s) {
  hipLaunchKernelGGL(slot_lens_kernel, dim3((uint32_t)((n + 1 + 255) / 256)), dim3(256), 0, s,
                     table, slots, n, lens);
  return hipGetLastError();
}

hipError_t launch_slot_write(const Slot* table, const uint64_t* slots, uint64_t n,
                             const uint64_t* word_offsets, uint8_t* words, void* counts,
                             uint32_t count_bytes, uint64_t count_bias, uint64_t* docs,
                             Header* hdr, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(slot_write_kernel, dim3((uint32_t)((n + 255) / 256)), dim3(256), 0, s,
                     table, slots, n, word_offsets, words, counts, count_bytes, count_bias, docs,
                     hdr);
  return hipGetLastError();
}

hipError_t launch_export(const ExportParams& E, hipStream_t s) {
  uint32_t nb = (uint32_t)E.n_blocks;
  hipLaunchKernelGGL(export_count_kernel, dim3(nb), dim3(kExportBlock), 0, s, E);
  hipLaunchKernelGGL(export_scan_kernel, dim3(1), dim3(1024), 0, s, E);
  hipLaunchKernelGGL(export_write_kernel, dim3(nb), dim3(kExportBlock), 0, s, E);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// merge: insert the entries of one table
// ------------------------------------------------------------------------------------------
// Adds the entries of up to kMergeInputs tables to one table; block b belongs to the input
// whose first_block is the last one at or before it. (One launch per table cost a merge of 96
// small tables 96 launches of about 10 us each, most of them with a handful of workgroups.)
__global__ __launch_bounds__(256) void merge_insert_kernel(MergeBatch M, Slot* table, uint64_t mask,
                                                           uint64_t occ_limit, uint64_t key_mask,
                                                           Header* hdr, uint64_t* joint,
                                                           uint32_t C) {
  uint32_t x = 0;
  while (x + 1 < M.n && M.first_block[x + 1] <= blockIdx.x) ++x;
  const MergeInput& in = M.in[x];
  uint64_t e = (blockIdx.x - M.first_block[x]) * 256ull + threadIdx.x;
  if (e >= in.n) return;
  uint64_t a = in.word_offsets[e], b = in.word_offsets[e + 1];
  uint64_t len = b - a;
  uint64_t c = in.count_bytes == 4 ? (uint64_t)(int64_t)((const int32_t*)in.counts)[e]
                                   : (uint64_t)((const int64_t*)in.counts)[e];
  if (len == 0 || c == 0) return;
  const uint8_t* w = in.words + a;
  uint64_t h = kFnvOffset, lo = 0, hi = 0;
  if (len <= 16) {
    load_packed(w, (uint32_t)len, in.words + in.word_offsets[in.n], &lo, &hi);
    h = fnv_packed(lo, hi, (uint32_t)len);
  } else {
    for (uint64_t q = 0; q < len; ++q) h = fnv_step(h, fold_byte(w[q]));
  }
  uint64_t key = finish_key(h, key_mask);
  WordId id = len <= 16 && packable(lo, hi) ? short_id(lo, hi, 0) : long_id(w, len, 0);
  uint64_t slot = table_insert<false>(table, mask, key, id, c, hdr, occ_limit);
  if (joint && slot != ~0ull) add64(&joint[slot * C + in.column], c);
}

hipError_t launch_merge_insert(const MergeInput* in, uint32_t k, Slot* table, uint64_t mask,
                               uint64_t occ_limit, uint64_t key_mask, Header* hdr,
                               uint64_t* joint_counts, uint32_t n_columns, hipStream_t s) {
  return for_merge_batches(in, k, 256, [&](const MergeBatch& M, uint32_t blocks) {
    hipLaunchKernelGGL(merge_insert_kernel, dim3(blocks), dim3(256), 0, s, M, table, mask,
                       occ_limit, key_mask, hdr, joint_counts, n_columns);
    return hipGetLastError();
  });
}

// ------------------------------------------------------------------------------------------
// FNV-1a 64 of strings (checked against published test vectors)
// ------------------------------------------------------------------------------------------
__global__ void hash_words_kernel(const uint8_t* bytes, const uint64_t* off, uint64_t n,
                                  uint64_t* out) {
  uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x;
  if (i >= n) return;
  uint64_t h = kFnvOffset;
  for (uint64_t q = off[i]; q < off[i + 1]; ++q) h = fnv_step(h, fold_byte(bytes[q]));
  uint64_t lo = 0, hi = 0, len = off[i + 1] - off[i];
  if (len <= 16) {
    for (uint64_t q = 0; q < len; ++q) {
      uint64_t f = fold_byte(bytes[off[i] + q]);
      if (q < 8) lo |= f << (8 * q); else hi |= f << (8 * (q - 8));
    }
    // the packed path the counter takes must agree with the byte path
    if (fnv_packed(lo, hi, packed_len(lo, hi)) != h) h = 0;  // reported as 1: a mismatch shows
  }
  out[i] = finish_key(h, ~0ull);
}

hipError_t launch_hash_words(const uint8_t* bytes, const uint64_t* offsets, uint64_t n,
                             uint64_t* out, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(hash_words_kernel, dim3((uint32_t)((n + 255) / 256)), dim3(256), 0, s,
                     bytes, offsets, n, out);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// top-k distinctive words
// ------------------------------------------------------------------------------------------
// The rank of an entry: by (n_c + 1) / (n_R + 1), then n_c, then word bytes. Sorting happens in
// LDS on 16-bit indices of records held there; most comparisons read only the ratio in double
// precision, which decides when two ratios differ by more than its rounding (each has at most five
// roundings of 2^-53); closer ratios are compared exactly.
struct RankLds {
  double* q;      // (n_c + 1) / (n_R + 1); -1: no entry here (after every entry)
  uint64_t* nc;
  uint64_t* nr;
  uint64_t* head; // the word's first 8 bytes, the first byte highest
  uint32_t* e;    // entry
};
constexpr size_t kRankBytes = 8 + 8 + 8 + 8 + 4 + 2;  // a record and its 16-bit index
constexpr uint32_t kRankBins = 2048;

// First 8 bytes of entry e's word, the first byte highest, zero padded (words have no zeros). The
// word bytes are in the workspace, which goes on after them.
WC_DEV uint64_t word_head(const TopkParams& P, uint64_t e) {
  const uint64_t a = P.word_offsets[e], n = P.word_offsets[e + 1] - a;
  uint64_t h;
  __builtin_memcpy(&h, P.words + a, 8);
  if (n < 8) h &= (1ull << (8 * n)) - 1;
  return __builtin_bswap64(h);
}

// true when word a comes before word b (bytes, unsigned, a proper prefix first)
WC_DEV bool word_before(const TopkParams& P, uint64_t a, uint64_t b) {
  const uint64_t pa = P.word_offsets[a], la = P.word_offsets[a + 1] - pa;
  const uint64_t pb = P.word_offsets[b], lb = P.word_offsets[b + 1] - pb;
  const uint64_t m = la < lb ? la : lb;
  for (uint64_t q = 0; q < m; ++q) {
    const uint8_t x = P.words[pa + q], y = P.words[pb + q];
    if (x != y) return x < y;
  }
  return la < lb;
}

// The exact order of (nc, nr) pairs; 0 when both are equal.
WC_DEV int pair_order(uint64_t na, uint64_t ra, uint64_t nb, uint64_t rb) {
  const uint64_t x = na + 1, y = rb + 1, u = nb + 1, v = ra + 1;
  const uint64_t lh = __umul64hi(x, y), ll = x * y, rh = __umul64hi(u, v), rl = u * v;
  if (lh != rh) return lh > rh ? 1 : -1;
  if (ll != rl) return ll > rl ? 1 : -1;
  if (na != nb) return na > nb ? 1 : -1;
  return 0;
}

WC_DEV bool rank_before(const TopkParams& P, const RankLds& R, uint32_t a, uint32_t b) {
  const double qa = R.q[a], qb = R.q[b], d = qa - qb, tol = fmax(qa, qb) * 0x1p-48;
  if (d > tol) return true;
  if (d < -tol) return false;
  if (R.e[a] == kNoRank || R.e[b] == kNoRank) return false;
  const int o = pair_order(R.nc[a], R.nr[a], R.nc[b], R.nr[b]);
  if (o) return o > 0;
  const uint64_t ha = R.head[a], hb = R.head[b];
  if (ha != hb) return ha < hb;
  return word_before(P, R.e[a], R.e[b]);
}

// Keeps the best min(k, kRankSpan) of kRankSpan candidates of one corpus, sorted. Level 0 takes the
// vocabulary (chunk blockIdx.x of it) and adds up the corpus's tokens; a later level takes the kept
// runs of the level before (run r: in_len[r] ids at in[r * run]).
//
// Only candidates that can be among the k best are sorted: a histogram over the leading bits of
// the ratio gives the bin that the k-th best falls into, and what lies below it is dropped. (The
// bins follow the double's bits, which the exact order agrees with up to its rounding; the bin
// below is kept too.) The sort is bitonic over 16-bit indices, its size the power of two that
// holds what is left; partners less than 128 apart stay inside a wave (no barrier). Four corpora
// of 43,000 words, top 50: level 0 79 us with all 2,048 sorted, 24 with those in reach; a later
// level 44 and 22.
//
// (One workgroup per corpus inserting every entry into per-thread lists of k in device memory
// took 4.35 ms: four workgroups on 256 CUs and a dependent device read per comparison.)
template <bool kLevel0>
__global__ __launch_bounds__(1024) void topk_sort_kernel(TopkParams P, const uint32_t* in,
                                                         const uint32_t* in_len, uint32_t in_runs,
                                                         uint32_t run, uint32_t* out,
                                                         uint32_t* out_len) {
  extern __shared__ __align__(16) uint8_t s_dyn[];
  __shared__ uint64_t s_sum[16], s_tmp[16];
  __shared__ uint32_t s_bin[kRankBins];
  __shared__ uint32_t s_n, s_left, s_cut;
  RankLds R;  // kRankSpan records and one that stands for none
  R.q = (double*)s_dyn;
  R.nc = (uint64_t*)(R.q + kRankSpan + 1);
  R.nr = R.nc + kRankSpan + 1;
  R.head = R.nr + kRankSpan + 1;
  R.e = (uint32_t*)(R.head + kRankSpan + 1);
  uint16_t* s_i = (uint16_t*)(R.e + kRankSpan + 1);
  const uint32_t t = threadIdx.x, c = blockIdx.y;
  if (P.hdr->flags) return;
  const uint64_t V = P.hdr->n_entries;
  const uint64_t minc = P.min_count > 0 ? P.min_count : 1;
  const uint64_t first = (uint64_t)blockIdx.x * kRankSpan;
  const uint32_t keep = P.k < kRankSpan ? P.k : kRankSpan;
  if (kLevel0 && first >= V) {  // a chunk past the vocabulary
    if (t == 0) out_len[(uint64_t)c * gridDim.x + blockIdx.x] = 0;
    return;
  }
  if (t == 0) {
    s_n = 0;
    s_left = 0;
    s_cut = 0;
    R.e[kRankSpan] = kNoRank;
    R.q[kRankSpan] = -1.0;
  }
  for (uint32_t i = t; i < kRankBins; i += 1024) s_bin[i] = 0;
  __syncthreads();
  // bin of a ratio: 8 exponent bits around 1 (2^-128 .. 2^127) and 3 mantissa bits
  auto bin_of = [](double q) -> uint32_t {
    const int32_t b = (int32_t)(__double_as_longlong(q) >> 49) - ((1023 - 128) << 3);
    return (uint32_t)min(max(b, 0), (int32_t)kRankBins - 1);
  };
  uint64_t sum = 0;
  uint32_t bin[kRankSpan / 1024];
#pragma unroll
  for (uint32_t x = 0; x < kRankSpan / 1024; ++x) {
    const uint32_t i = t + x * 1024;
    uint32_t e = kNoRank;
    if (kLevel0) {
      if (first + i < V) e = (uint32_t)(first + i);
    } else {
      const uint64_t at = first + i;
      const uint32_t r = (uint32_t)(at / run), j = (uint32_t)(at - (uint64_t)r * run);
      if (r < in_runs && j < in_len[(uint64_t)c * in_runs + r])
        e = in[(uint64_t)c * in_runs * run + at];
    }
    uint64_t nc = 0, nr = 0;
    if (e != kNoRank) {
      nc = P.joint[P.slot_of_entry[e] * P.C + c];
      nr = P.entry_total[e] - nc;
      sum += nc;
      if (nc < minc) e = kNoRank;
    }
    R.e[i] = e;
    R.nc[i] = nc;
    R.nr[i] = nr;
    const double q = e == kNoRank ? -1.0 : ((double)nc + 1.0) / ((double)nr + 1.0);
    R.q[i] = q;
    bin[x] = bin_of(q);
    if (e != kNoRank) atomicAdd(&s_bin[bin[x]], 1u);
    const uint64_t m = __ballot(e != kNoRank);
    if ((t & 63) == 0 && m) atomicAdd(&s_n, (uint32_t)__popcll(m));
  }
  if (kLevel0) {
    for (int d = 32; d >= 1; d >>= 1) sum += __shfl_xor(sum, d, 64);
    if ((t & 63) == 0) s_sum[t >> 6] = sum;
  }
  __syncthreads();
  if (kLevel0 && t == 0) {
    uint64_t s = 0;
    for (int w = 0; w < 16; ++w) s += s_sum[w];
    if (s) add64(&P.totals[c], s);
  }
  // the highest bin at which at least `keep` candidates lie in it and above (thread t: bins
  // 2 t' and 2 t' + 1 from the top)
  {
    const uint32_t hi = kRankBins - 1 - 2 * t;
    const uint32_t a = s_bin[hi], b = s_bin[hi - 1];
    uint64_t tot;
    const uint32_t above = (uint32_t)block_excl_scan<1024>(a + b, s_tmp, &tot);
    if (above < keep && above + a + b >= keep) s_cut = above + a >= keep ? hi : hi - 1;
  }
  __syncthreads();
  const uint32_t cut = s_cut ? s_cut - 1 : 0u;
#pragma unroll
  for (uint32_t x = 0; x < kRankSpan / 1024; ++x) {
    const uint32_t i = t + x * 1024, e = R.e[i];
    const bool in_reach = e != kNoRank && bin[x] >= cut;
    const uint64_t m = __ballot(in_reach);
    uint32_t base = 0;
    if ((t & 63) == 0 && m) base = atomicAdd(&s_left, (uint32_t)__popcll(m));
    base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
    if (in_reach) {
      s_i[base + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                           __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))] = (uint16_t)i;
      R.head[i] = word_head(P, e);
    }
  }
  __syncthreads();
  const uint32_t left = s_left;
  uint32_t span = 128;  // (a wave's worth of pairs at least)
  while (span < left) span <<= 1;
  for (uint32_t i = left + t; i < span; i += 1024) s_i[i] = (uint16_t)kRankSpan;
  __syncthreads();
  for (uint32_t size = 2; size <= span; size <<= 1) {
    for (uint32_t j = size >> 1; j; j >>= 1) {
      const uint32_t i = ((t & ~(j - 1)) << 1) | (t & (j - 1)), l = i + j;
      if (t < span / 2) {
        const uint32_t a = s_i[i], b = s_i[l];
        if (rank_before(P, R, b, a) == ((i & size) == 0)) {
          s_i[i] = (uint16_t)b;
          s_i[l] = (uint16_t)a;
        }
      }
      // a wave's 64 pairs at distance j <= 64 lie in its own 128 elements, and so do those of
      // the next stage unless it starts a size above 128
      const bool local = j > 1 ? j <= 64 : size < 128;
      if (local) {
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __builtin_amdgcn_wave_barrier();
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
      } else {
        __syncthreads();
      }
    }
  }
  __syncthreads();
  const uint32_t n = min(s_n, keep);
  uint32_t* o = out + ((uint64_t)c * gridDim.x + blockIdx.x) * keep;
  for (uint32_t i = t; i < n; i += 1024) o[i] = R.e[s_i[i]];
  if (t == 0) out_len[(uint64_t)c * gridDim.x + blockIdx.x] = n;
}

// For k above half of kRankSpan: pairs of sorted runs merged, each id to the place that its own
// position and the number of better ids of the other run give (a binary search); the best k stay.
// (Pairs in x: the other dimensions of a grid end at 65,535.)
__global__ __launch_bounds__(256) void topk_merge_kernel(TopkParams P, const uint32_t* in,
                                                         const uint32_t* in_len, uint32_t in_runs,
                                                         uint32_t run, uint32_t* out,
                                                         uint32_t* out_len, uint32_t out_run) {
  const uint32_t c = blockIdx.z, pair = blockIdx.x, out_runs = gridDim.x;
  if (P.hdr->flags) return;
  const uint32_t at = blockIdx.y * 256 + threadIdx.x;  // position among both runs
  const uint32_t side = at / run, i = at - side * run;
  if (side > 1) return;
  const uint64_t base = (uint64_t)c * in_runs;
  const uint32_t mine = 2 * pair + side, other = 2 * pair + 1 - side;
  const uint32_t nm = mine < in_runs ? in_len[base + mine] : 0u;
  const uint32_t no = other < in_runs ? in_len[base + other] : 0u;
  if (at == 0) out_len[(uint64_t)c * out_runs + pair] = min(nm + no, P.k);
  if (i >= nm) return;
  const uint32_t* A = in + (base + mine) * run;
  const uint32_t* B = in + (base + other) * run;
  const uint64_t e = A[i];
  const uint64_t na = P.joint[P.slot_of_entry[e] * P.C + c], ra = P.entry_total[e] - na;
  uint32_t lo = 0, hi = no;  // ids of the other run before this one
  while (lo < hi) {
    const uint32_t m = (lo + hi) >> 1;
    const uint64_t f = B[m];
    const uint64_t nb = P.joint[P.slot_of_entry[f] * P.C + c], rb = P.entry_total[f] - nb;
    const int o = pair_order(na, ra, nb, rb);
    if (o < 0 || (o == 0 && word_before(P, f, e))) lo = m + 1;
    else hi = m;
  }
  const uint32_t rank = i + lo;
  if (rank < P.k) out[((uint64_t)c * out_runs + pair) * out_run + rank] = (uint32_t)e;
}

// Rows of the answer, their word offsets and bytes (one workgroup), and the sizes the host reads.
__global__ __launch_bounds__(1024) void topk_rows_kernel(TopkParams P, const uint32_t* best,
                                                         const uint32_t* best_len, uint32_t run) {
  __shared__ uint64_t s_tmp[16];
  __shared__ uint64_t s_carry;
  if (threadIdx.x == 0) {
    s_carry = 0;
    P.sizes->flags = P.hdr->flags;
    P.sizes->vocab = P.hdr->n_entries;
  }
  if (P.hdr->flags) return;
  const uint64_t V = P.hdr->n_entries;
  uint64_t all = 0;
  for (uint32_t q = 0; q < P.C; ++q) all += P.totals[q];
  if (threadIdx.x < P.C) P.sizes->n_rows[threadIdx.x] = best_len[threadIdx.x];
  __syncthreads();
  const uint64_t total_rows = (uint64_t)P.C * P.k;
  for (uint64_t base = 0; base < total_rows; base += 1024) {
    const uint64_t r = base + threadIdx.x;
    uint64_t len = 0, e = 0;
    if (r < total_rows) {
      const uint32_t c = (uint32_t)(r / P.k), j = (uint32_t)(r % P.k);
      if (j < best_len[c]) {
        e = best[(uint64_t)c * run + j];
        len = P.word_offsets[e + 1] - P.word_offsets[e];
        const uint64_t nc = P.joint[P.slot_of_entry[e] * P.C + c], nr = P.entry_total[e] - nc;
        const double Nc = (double)P.totals[c], Nr = (double)(all - P.totals[c]), Vd = (double)V;
        P.out_nc[r] = nc;
        P.out_nr[r] = nr;
        P.out_score[r] = (((double)nc + 1.0) / (Nc + Vd)) / (((double)nr + 1.0) / (Nr + Vd));
      }
    }
    uint64_t tot;
    const uint64_t ex = block_excl_scan<1024>(len, s_tmp, &tot);
    const uint64_t pos = ex + s_carry;
    if (r < total_rows) {
      P.out_word_offsets[r] = pos;
      const uint8_t* src = P.words + P.word_offsets[e];
      for (uint64_t q = 0; q < len; ++q) P.out_words[pos + q] = src[q];
    }
    __syncthreads();
    if (threadIdx.x == 0) s_carry += tot;
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    P.out_word_offsets[total_rows] = s_carry;
    P.sizes->word_bytes = s_carry;
  }
}

// ids (and run lengths) that one of the two list buffers holds at most for `n` vocabulary words
uint64_t topk_list_ids(uint64_t n, uint32_t k) {
  return ((n + kRankSpan - 1) / kRankSpan + 1) * (k < kRankSpan ? k : kRankSpan) + k;
}
uint64_t topk_list_runs(uint64_t n) { return (n + kRankSpan - 1) / kRankSpan + 1; }

// The vocabulary's size is on the device; `n` bounds it, so that no host wait comes between the
// joint table and the ranking (chunks past the vocabulary keep nothing).
hipError_t launch_topk(const TopkParams& P, uint64_t n, hipStream_t s) {
  static const hipError_t attr = [] {
    hipError_t e = hipFuncSetAttribute((const void*)topk_sort_kernel<true>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)((kRankSpan + 1) * kRankBytes));
    if (e == hipSuccess)
      e = hipFuncSetAttribute((const void*)topk_sort_kernel<false>,
                              hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)((kRankSpan + 1) * kRankBytes));
    return e;
  }();
  if (attr != hipSuccess) return attr;
  const size_t dyn = (kRankSpan + 1) * kRankBytes;
  uint32_t runs = (uint32_t)((n + kRankSpan - 1) / kRankSpan);
  if (runs == 0) runs = 1;
  uint32_t run = P.k < kRankSpan ? P.k : kRankSpan;
  hipLaunchKernelGGL(topk_sort_kernel<true>, dim3(runs, P.C), dim3(1024), dyn, s, P, nullptr,
                     nullptr, 0u, 1u, P.lists[0], P.list_len[0]);
  int src = 0;
  while (runs > 1) {
    const int dst = src ^ 1;
    if (P.k <= kRankSpan / 2) {  // a level keeps at most half of what it sorts
      const uint32_t next = (uint32_t)(((uint64_t)runs * run + kRankSpan - 1) / kRankSpan);
      hipLaunchKernelGGL(topk_sort_kernel<false>, dim3(next, P.C), dim3(1024), dyn, s, P,
                         P.lists[src], P.list_len[src], runs, run, P.lists[dst], P.list_len[dst]);
      runs = next;
    } else {
      const uint32_t next = (runs + 1) / 2;
      const uint32_t longer = 2 * run < P.k ? 2 * run : P.k;
      hipLaunchKernelGGL(topk_merge_kernel, dim3(next, (2 * run + 255) / 256, P.C), dim3(256), 0,
                         s, P, P.lists[src], P.list_len[src], runs, run, P.lists[dst],
                         P.list_len[dst], longer);
      runs = next;
      run = longer;
    }
    src = dst;
  }
  hipLaunchKernelGGL(topk_rows_kernel, dim3(1), dim3(1024), 0, s, P, P.lists[src],
                     P.list_len[src], run);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// ------------------------------------------------------------------------------------------
// exclusive prefix sum of uint64 values: per-block scans, a scan of the block totals, and
// the block offsets added back
// ------------------------------------------------------------------------------------------
constexpr uint32_t kScanBlock = 256, kScanItems = 4, kScanSpan = kScanBlock * kScanItems;

uint64_t excl_scan_scratch(uint64_t n) { return ((n + kScanSpan - 1) / kScanSpan + 1) * 8; }

// out[i] = sum of in[b*span .. i) for the block b holding i; sums[b] = the block's total
__global__ __launch_bounds__(kScanBlock) void scan_local_kernel(const uint64_t* in, uint64_t* out,
                                                                uint64_t n, uint64_t* sums) {
  __shared__ uint64_t s_tmp[kScanBlock / 64];
  const uint64_t first = blockIdx.x * (uint64_t)kScanSpan + (uint64_t)threadIdx.x * kScanItems;
  uint64_t v[kScanItems], t = 0;
  for (uint32_t j = 0; j < kScanItems; ++j) {
    v[j] = first + j < n ? in[first + j] : 0;
    t += v[j];
  }
  uint64_t tot;
  uint64_t e = block_excl_scan<kScanBlock>(t, s_tmp, &tot);
  for (uint32_t j = 0; j < kScanItems; ++j) {
    if (first + j < n) out[first + j] = e;
    e += v[j];
  }
  if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

// sums[0 .. nb) becomes its exclusive scan (one workgroup)
__global__ __launch_bounds__(1024) void scan_sums_kernel(uint64_t* sums, uint64_t nb) {
  __shared__ uint64_t s_tmp[16];
  __shared__ uint64_t s_carry;
  if (threadIdx.x == 0) s_carry = 0;
  __syncthreads();
  for (uint64_t base = 0; base < nb; base += 1024) {
    const uint64_t i = base + threadIdx.x;
    const uint64_t v = i < nb ? sums[i] : 0;
    uint64_t tot;
    const uint64_t e = block_excl_scan<1024>(v, s_tmp, &tot);
    if (i < nb) sums[i] = e + s_carry;
    __syncthreads();
    if (threadIdx.x == 0) s_carry += tot;
    __syncthreads();
  }
}

__global__ void scan_add_kernel(uint64_t* out, uint64_t n, const uint64_t* sums) {
  const uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x;
  if (i < n) out[i] += sums[i / kScanSpan];
}

hipError_t excl_scan_u64(const uint64_t* in, uint64_t* out, uint64_t n, uint64_t* sums,
                         hipStream_t s) {
  if (n == 0) return hipSuccess;
  const uint64_t nb = (n + kScanSpan - 1) / kScanSpan;
  hipLaunchKernelGGL(scan_local_kernel, dim3((uint32_t)nb), dim3(kScanBlock), 0, s, in, out, n,
                     sums);
  if (nb > 1) {
    hipLaunchKernelGGL(scan_sums_kernel, dim3(1), dim3(1024), 0, s, sums, nb);
    hipLaunchKernelGGL(scan_add_kernel, dim3((uint32_t)((n + 255) / 256)), dim3(256), 0, s, out,
                       n, sums);
  }
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// entries grouped by document: a counting sort (histogram, scan, scatter); the order inside a
// document is unspecified, as the result's entry order is
// ------------------------------------------------------------------------------------------
__global__ void doc_hist_kernel(const uint64_t* docs, uint64_t n, uint64_t* doc_len) {
  const uint64_t e = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x;
  if (e < n) atomicAdd((unsigned long long*)&doc_len[docs[e]], 1ull);
}

__global__ void doc_scatter_kernel(const uint64_t* docs, const uint64_t* slots, uint64_t n,
                                   const uint64_t* doc_ptr, uint64_t* fill,
                                   uint64_t* sorted_docs, uint64_t* sorted_slots) {
  const uint64_t e = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x;
  if (e >= n) return;
  const uint64_t d = docs[e];
  const uint64_t at = doc_ptr[d] + atomicAdd((unsigned long long*)&fill[d], 1ull);
  sorted_docs[at] = d;
  sorted_slots[at] = slots[e];
}

hipError_t group_by_doc(const uint64_t* docs, const uint64_t* slots, uint64_t n, uint64_t n_docs,
                        uint64_t* doc_ptr, uint64_t* doc_len, uint64_t* fill, uint64_t* sums,
                        uint64_t* sorted_docs, uint64_t* sorted_slots, hipStream_t s) {
  hipError_t e = launch_fill_zero(doc_len, n_docs * 8, s);
  if (e == hipSuccess) e = launch_fill_zero(fill, n_docs * 8, s);
  if (e != hipSuccess || n_docs == 0) return e;
  const uint32_t grid = (uint32_t)((n + 255) / 256);
  if (n) hipLaunchKernelGGL(doc_hist_kernel, dim3(grid), dim3(256), 0, s, docs, n, doc_len);
  e = excl_scan_u64(doc_len, doc_ptr, n_docs, sums, s);
  if (e == hipSuccess && n)
    hipLaunchKernelGGL(doc_scatter_kernel, dim3(grid), dim3(256), 0, s, docs, slots, n, doc_ptr,
                       fill, sorted_docs, sorted_slots);
  return e == hipSuccess ? hipGetLastError() : e;
}

}  // namespace wc
