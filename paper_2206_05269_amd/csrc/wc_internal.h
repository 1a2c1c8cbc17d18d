// Internal interfaces between the host API (wc_api.hip) and the kernel files.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/wc.h"
#include "wc_device.h"

namespace wc {

struct CountParams {
  const uint8_t* corpus;     // logical byte 0
  uint64_t len;
  const uint64_t* offsets;   // [n_docs + 1]
  uint64_t n_docs;
  uint64_t R0, R1;           // offsets[0], offsets[n_docs] (host copies)
  Slot* table;
  uint64_t mask;             // slots - 1
  uint64_t occ_limit;        // claimed slots above this set the full flag
  uint64_t key_mask;
  Header* hdr;
  const uint64_t* stage_doc; // [n_stages + 1]
  int64_t base_off;          // logical position of stage 0 (<= 0, > -16)
  uint64_t n_stages;
  uint64_t stages_per_wg;
  uint32_t lds_entries;
  uint32_t lds_flush_at;
  uint32_t policy;
  uint32_t no_lds;
  uint32_t utf8;             // WC_TOKENIZE_UTF8: the UTF-8 reading of word bytes
  uint32_t pad0;
};

// two-pass global count (wc_global.hip)
constexpr uint32_t kParts = 256;         // partitions of the spilled records
constexpr uint32_t kBlockRec = 256;      // records per arena block (4 KiB)
constexpr uint32_t kDictMax = 5120;      // hot-word dictionary capacity (words)
constexpr uint32_t kMapBlock = 1024;     // pass-1 workgroup
constexpr uint32_t kGlobalStage = kMapBlock * 16;  // bytes scanned per pass-1 stage
constexpr uint32_t kDispBuckets = 1024;   // dictionary: displacement buckets (low 9 hash bits)
constexpr uint32_t kDictSlots = 8192;    // dictionary: slots of the perfect hash
constexpr uint32_t kDictRegions = 32;    // dictionary: regions of 256 slots (group mod 32)
constexpr uint32_t kSampleStages = 512;  // pass-1 stages sampled (first 8 KiB of each)
constexpr uint32_t kSamplePer = 2;       // sampled stages per sample workgroup
constexpr uint32_t kSampleLds = 2048;    // LDS table of one sample workgroup
constexpr uint64_t kSampleSlots = 1ull << 19;  // device table of the sample
constexpr uint32_t kStripe = 1024;       // pass-1 bytes per wave per stage
constexpr uint32_t kStripeText = 16 + kStripe + 16;  // per wave: prefix, stripe, padding
constexpr uint32_t kWaveStarts = 192;    // word starts of one wave listed at a time
constexpr uint32_t kDictCols = 64;       // dictionary words totalled per pass-2 workgroup
constexpr uint32_t kWinBlocks = 2048;    // pass 2 lists the non-empty blocks this many at a time
constexpr uint32_t kRedSlots = 8192;     // pass-2 LDS slots (13-bit entry indices)

// Dictionary of hot words, chosen from a sample and read-only while the text is scanned: a
// perfect hash by hash-and-displace. A word with hash h belongs to group h mod 512; the group's
// displacement picks its slot in region (h mod 16) (see dict_slot); the slot holds its key
// index; empty slots hold n, the index of an all-zero key that no word matches.
struct DictImage {
  uint32_t n;            // words (key entries) in the dictionary
  uint32_t placed;       // words placed in the perfect hash (the others are never looked up)
  uint32_t n_high;       // selection: words above the count threshold
  uint32_t n_low;        // selection: words at the threshold competing for the rest
  uint32_t hist[256];    // sample counts (clamped at 255) -> number of words
  uint16_t disp[kDispBuckets];
  uint16_t slot[kDictSlots];
  uint4 keys[kDictMax + 1];  // packed words (lo, hi); keys[n] = 0
  uint32_t cnt[kDictMax];    // their sample counts (clamped at 255)
};

struct GlobalParams {
  const uint8_t* corpus;
  uint64_t len;
  const uint64_t* offsets;
  uint64_t n_docs;
  Slot* table;
  uint64_t mask;
  uint64_t occ_limit;
  uint64_t key_mask;
  Header* hdr;
  const uint64_t* stage_doc;
  int64_t base_off;
  uint64_t n_stages;
  uint64_t stages_per_wg;
  uint32_t map_grid;         // pass-1 workgroups
  uint32_t dict_cap;         // dictionary capacity (<= kDictMax)
  DictImage* dict;
  uint32_t* dict_part;       // [map_grid][dict_cap] dictionary hits per pass-1 workgroup
  Slot* sample_table;        // [kSampleSlots]
  Header* sample_hdr;
  uint32_t reduce_entries;   // pass-2 LDS entries (distinct words of a partition, <= kRedSlots)
  uint32_t reduce_cap;       // entries used before further new words go to the global table
  uint32_t S;                // blocks per partition (kParts * S < 2^32): block k = w * J + j is
                             // the j-th of pass-1 workgroup w (J = S / map_grid)
  uint4* arena;              // [S][kParts][kBlockRec] records: block k of partition p at k * kParts + p
  uint16_t* fill;            // [kParts][S] records per block (zero before pass 1)
};
size_t global_map_dyn(uint32_t dict_cap);
size_t global_reduce_dyn(uint32_t entries);
hipError_t set_global_smem(uint32_t dict_cap, uint32_t reduce_entries);
// Sample, dictionary, pass 1 (between events a and b when given) and pass 2. The sample
// table, its header, the dictionary image and the block fills must be zero.
hipError_t launch_global(const GlobalParams& P, hipEvent_t a, hipEvent_t b, hipStream_t s);

// partitioned global count (wc_part.hip)
constexpr uint32_t kPartMapEntries = 5008;  // LDS entries of a map workgroup (20 bytes each)
constexpr uint32_t kPartRedEntries = 5888;  // of a reduce workgroup
constexpr uint32_t kPartMergeEntries = 5056;  // of a merge's reduce workgroup (24 bytes each)
struct PartParams {
  const uint8_t* corpus;
  uint64_t len;
  const uint64_t* offsets;
  uint64_t n_docs;
  Header* hdr;               // zero before the map
  int64_t base_off;          // logical position of stripe 0 (<= 0, > -16)
  uint64_t n_stripes;
  uint64_t stripes_per_wg;
  uint32_t parts;            // partitions: a power of two, at most kParts
  uint32_t max_lists;
  uint64_t cap_recs;
  uint4* rec_key;            // [cap_recs] a word of a list ...
  void* rec_cnt;             // [cap_recs] ... and its count in it (uint32_t; merge: uint64_t)
  uint2* dir;                // [parts][max_lists] first record and records of a list's partition
  uint64_t* word_offsets;    // [slots + 1]
  uint8_t* words;            // [word_cap]
  void* counts;              // [slots]
  uint64_t slots, occ_limit, word_cap;
  uint64_t count_bias;
  uint32_t count_bytes;
  uint32_t utf8;             // WC_TOKENIZE_UTF8: the UTF-8 reading of word bytes
};
hipError_t set_part_smem();
hipError_t launch_part_map(const PartParams& P, uint32_t grid, hipStream_t s);
hipError_t launch_part_reduce(const PartParams& P, hipStream_t s);
// a text that one workgroup counts and writes by itself (clears the header too)
hipError_t launch_part_single(const PartParams& P, hipStream_t s);

// per-document count (wc_docs.hip)
constexpr uint64_t kMinWin = 16 * 1024, kMaxWin = 48 * 1024;  // bytes per work item
constexpr uint32_t kDirectKib = 72;
// Work items by their bytes: class 0 below 16 KiB, class k from 8 KiB << k on.
constexpr uint32_t kDocClasses = 16;
constexpr uint32_t kDocW = 256;        // documents per sub-window
constexpr uint32_t kDocSlots = 8192;   // LDS table slots
constexpr uint32_t kDocLds = 4628;     // LDS table entries (20 bytes each, beside 8192 slots)

struct DocTask {           // device-resident: every size the per-document kernels read
  const uint8_t* corpus;
  uint64_t len;
  const uint64_t* offsets;
  uint64_t n_docs;
};

struct DocParams {
  const DocTask* task;
  Header* hdr;
  uint64_t* items;         // runs of documents, by size class
  uint64_t class_at[kDocClasses + 1];  // a class's first item, and where the last one's end at most
  uint32_t* class_n;       // [kDocClasses] items of each class (zero before)
  uint64_t* word_offsets;  // [cap_e + 1]
  uint8_t* words;          // [cap_b]
  void* counts;
  uint32_t count_bytes;
  uint32_t grid;           // workgroups
  uint32_t lds_cap;        // entries used before keys are spilled
  uint32_t direct_kib;     // documents above this many KiB, and a window, are reported (0: none)
  uint64_t win_bytes;      // work item window; 0: by the size of the text
  uint64_t* docs;          // [cap_e]
  uint64_t* doc_ptr;       // [n_docs]
  uint64_t* doc_len;       // [n_docs]
  uint64_t cap_e, cap_b;
  Slot* arena;             // spilled keys and tables set aside
  uint64_t arena_slots;
  uint64_t count_bias;     // added to every exported count (debug; 0 normally)
};
hipError_t set_doc_smem();
constexpr size_t kDocHeadBytes = sizeof(Header) + kDocClasses * 4;  // the header and class_n
// clears them and sets the task
hipError_t launch_doc_begin(Header* hdr, DocTask* task, const DocTask& value, hipStream_t s);
hipError_t launch_docs(const DocParams& P, hipStream_t s);

hipError_t launch_count(const CountParams& P, bool per_doc, uint32_t grid, uint32_t block,
                        size_t dyn, hipStream_t s);
hipError_t set_count_smem(uint32_t block, size_t dyn);
hipError_t launch_stage_doc(const uint64_t* offsets, uint64_t n_docs, int64_t base_off,
                            uint32_t stage, uint64_t n_stages, uint64_t* out, hipStream_t s);
hipError_t launch_validate(const uint64_t* offsets, uint64_t n_docs, uint64_t len, Header* hdr,
                           hipStream_t s);

// ---- export (compaction of a table into dense arrays) -----------------------------------
struct ExportParams {
  const Slot* table;
  uint64_t slots;
  Header* hdr;
  uint64_t* block_sums;      // [2 * n_blocks] (entries, bytes) per block, then scanned
  uint64_t n_blocks;
  uint64_t* word_offsets;    // [slots + 1]
  uint8_t* words;
  uint64_t word_cap;
  void* counts;
  uint32_t count_bytes;
  uint32_t per_doc;
  uint64_t* docs;            // per-document: entry document
  uint64_t* slot_of_entry;   // optional: entry -> slot (joint tables)
  uint64_t* entry_of_slot;   // optional: slot -> entry
  uint64_t count_bias;       // added to every exported count (debug; 0 normally)
};
constexpr uint32_t kExportBlock = 256;
constexpr uint32_t kExportItems = 4;  // slots per thread
constexpr uint64_t kExportSpan = kExportBlock * kExportItems;

hipError_t launch_export(const ExportParams& E, hipStream_t s);
hipError_t launch_export_list(const ExportParams& E, hipStream_t s);
hipError_t launch_slot_lens(const Slot* table, const uint64_t* slots, uint64_t n, uint64_t* lens,
                            hipStream_t s);
hipError_t launch_slot_write(const Slot* table, const uint64_t* slots, uint64_t n,
                             const uint64_t* word_offsets, uint8_t* words, void* counts,
                             uint32_t count_bytes, uint64_t count_bias, uint64_t* docs,
                             Header* hdr, hipStream_t s);
// exclusive prefix sum of n uint64 values (out may be in); sums: excl_scan_scratch(n) bytes
uint64_t excl_scan_scratch(uint64_t n);
hipError_t excl_scan_u64(const uint64_t* in, uint64_t* out, uint64_t n, uint64_t* sums,
                         hipStream_t s);
// entries (docs[e], slots[e]) grouped by document into sorted_*; doc_ptr / doc_len per
// document; fill: n_docs scratch; sums: excl_scan_scratch(n_docs)
hipError_t group_by_doc(const uint64_t* docs, const uint64_t* slots, uint64_t n, uint64_t n_docs,
                        uint64_t* doc_ptr, uint64_t* doc_len, uint64_t* fill, uint64_t* sums,
                        uint64_t* sorted_docs, uint64_t* sorted_slots, hipStream_t s);

// ---- fills ---------------------------------------------------------------------------------
hipError_t launch_fill_zero(void* p, uint64_t bytes, hipStream_t s);

// ---- merge ---------------------------------------------------------------------------------
struct MergeInput {
  const uint64_t* word_offsets;
  const uint8_t* words;
  const void* counts;
  uint64_t n;
  uint32_t count_bytes;
  uint32_t column;           // joint tables: column of this input
};
constexpr uint32_t kMergeInputs = 32;  // tables one launch adds (they are kernel arguments)
struct MergeBatch {
  MergeInput in[kMergeInputs];
  uint32_t first_block[kMergeInputs];
  uint32_t n;
};
// launch(batch, workgroups) for the inputs, kMergeInputs at a time, `span` entries per workgroup
// (of at most 1,024 threads; a launch has fewer than 2^32 threads, so many large inputs take several)
constexpr uint64_t kMergeBlocks = 0xffffffffull / 1024;
template <class Launch>
hipError_t for_merge_batches(const MergeInput* in, uint32_t k, uint32_t span, Launch launch) {
  for (uint32_t i = 0; i < k;) {
    MergeBatch M;
    uint64_t blocks = 0;
    for (M.n = 0; i < k && M.n < kMergeInputs; ++i) {
      const uint64_t nb = (in[i].n + span - 1) / span;
      if (nb == 0) continue;
      if (blocks + nb > kMergeBlocks && M.n) break;
      M.in[M.n] = in[i];
      M.first_block[M.n++] = (uint32_t)blocks;
      blocks += nb;
    }
    if (M.n == 0) continue;
    const hipError_t e = launch(M, (uint32_t)blocks);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}
hipError_t launch_merge_insert(const MergeInput* in, uint32_t k, Slot* table, uint64_t mask,
                               uint64_t occ_limit, uint64_t key_mask, Header* hdr,
                               uint64_t* joint_counts, uint32_t n_columns, hipStream_t s);

// merge through hash partitions (wc_part.hip): the inputs' entries as records, then the reduce.
// The header must be zero; arena for all entries (64-bit counts), a list per kMergeSpan of an input.
constexpr uint32_t kMergeSpan = 4096;
hipError_t launch_part_merge(const MergeInput* in, uint32_t k, const PartParams& P, hipStream_t s);

// ---- dense reduce (the zero-padded keys x documents matrix) --------------------------------
hipError_t launch_dense_keys(const MergeInput& in, Slot* table, uint64_t mask,
                             uint64_t occ_limit, uint64_t key_mask, Header* hdr,
                             uint64_t* slot_of_input, hipStream_t s);
hipError_t launch_dense_scatter(uint64_t n, const uint64_t* slot_of_input,
                                const uint64_t* entry_of_slot, const uint64_t* docs,
                                const void* counts, uint32_t count_bytes, uint64_t n_docs,
                                uint32_t* matrix, hipStream_t s);
hipError_t launch_dense_rowsum(const uint32_t* matrix, uint64_t rows, uint64_t n_docs,
                               void* counts, uint32_t count_bytes, uint64_t bias, Header* hdr,
                               hipStream_t s);

// ---- top-k ---------------------------------------------------------------------------------
struct TopkSizes {               // what the host reads back
  uint64_t n_rows[64];
  uint64_t word_bytes, vocab, flags;
};
struct TopkParams {
  const Header* hdr;             // of the joint table: vocabulary size, flags
  const uint64_t* word_offsets;  // joint vocabulary, V entries
  const uint8_t* words;
  const uint64_t* joint;         // [slots * C] counts per slot and corpus
  const uint64_t* slot_of_entry; // [V]
  const uint64_t* entry_total;   // [V] sum over corpora
  uint32_t C;
  uint32_t k;
  uint64_t min_count;
  uint64_t* totals;              // [C] token totals per corpus (zero before launch_topk)
  uint32_t* lists[2];            // scratch: [C * topk_list_ids] kept ids of a level
  uint32_t* list_len[2];         // scratch: [C * topk_list_runs]
  TopkSizes* sizes;
  // outputs
  uint64_t* out_word_offsets;    // [C*k + 1]
  uint8_t* out_words;
  uint64_t* out_nc;
  uint64_t* out_nr;
  double* out_score;
};
constexpr uint32_t kRankSpan = 2048;         // candidates one workgroup sorts
constexpr uint32_t kNoRank = 0xffffffffu;
uint64_t topk_list_ids(uint64_t n, uint32_t k);
uint64_t topk_list_runs(uint64_t n);
hipError_t launch_topk(const TopkParams& P, uint64_t n, hipStream_t s);

// ---- hashing (debug entry point) ------------------------------------------------------------
hipError_t launch_hash_words(const uint8_t* bytes, const uint64_t* offsets, uint64_t n,
                             uint64_t* out, hipStream_t s);

}  // namespace wc
