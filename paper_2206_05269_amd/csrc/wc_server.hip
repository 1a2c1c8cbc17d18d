// Serving: a request loop that counts texts as they arrive, keeps the resulting tables
// resident on the device and answers merge queries (Section 3.3's summation of grouped counts,
// across requests).
//
// Admission. The server owns one device pool of `mem_budget` bytes; the policy (count memory
// from the low end, resident tables from the high end, in order, when to wait and when to fail) is the
// host-only wc::Admission of wc_admission.h. A request is admitted when the memory its count
// needs (text, offsets, workspace) is free; until then it waits in arrival order. Results are
// compacted into an exact-size resident block, and the count memory is returned at once.
//
// Continuous batching. `max_streams` worker threads each own a HIP stream (default priority),
// so admitted requests run concurrently on the device. A worker that takes a small
// single-document request also takes the small single-document requests queued right behind
// it (up to kPackDocs requests) and counts them in one per-document launch, then splits the
// per-document tables into one resident table per request: one kernel gathers the group's texts,
// one finds every request's entries, bytes and tokens, and one copies all their tables, with a
// host wait after the second and the third. Requests above kSmallBytes are counted alone: the
// partitioned count takes 42 us and up, text in device memory is read where it is, and the table
// goes to its resident block with one launch. (Requests of up to 1 MiB used to be packed and
// split one at a time, with two host waits and three copies each: 96 requests of 1 KiB to 4 MiB and
// a merge of their tables took 5.8 ms.)
//
// Uploads. Each worker owns two pinned host buffers: it copies a request's text into one while
// the other is on its way to the device, so host copies of several workers and their DMA
// transfers overlap (a copy straight from pageable memory goes through the runtime's own
// staging, one transfer at a time).
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <condition_variable>
#include <deque>
#include <map>
#include <memory>
#include <mutex>
#include <thread>
#include <unordered_map>
#include <vector>

#include "wc_admission.h"
#include "wc_internal.h"

namespace {

using Clock = std::chrono::steady_clock;

constexpr uint32_t kPackDocs = 64;
constexpr uint64_t kSmallBytes = 32ull << 10;
constexpr uint64_t kStageBytes = 8ull << 20;  // per pinned upload buffer (two per worker)

struct Request {
  uint64_t id = 0;
  std::vector<uint8_t> text;      // host copy (host input)
  const uint8_t* dev_text = nullptr;
  const uint8_t* host_text = nullptr;  // caller's host memory, read in place (not copied)
  uint64_t len = 0;
  std::vector<uint64_t> offsets;
  wc_opts opts{};
  wc_tuning tuning{};
  bool merge = false;
  std::vector<uint64_t> merge_ids;
  // state
  std::vector<std::shared_ptr<Request>> merge_inputs;  // pinned at submission
  int state = 0;  // 0 queued, 1 running, 2 done
  wc_status status = WC_EAGAIN;
  uint8_t* resident = nullptr;
  wc::ResidentLife life;  // merges reading the resident table; released by the client
  wc_result res{};
  double t_submit = 0, t_start = 0, t_done = 0;
};

double now_s() {
  return std::chrono::duration<double>(Clock::now().time_since_epoch()).count();
}

}  // namespace

struct wc_server {
  int device = 0;
  uint64_t budget = 0;
  uint8_t* pool_mem = nullptr;
  wc::Admission adm;
  std::mutex mu;
  std::condition_variable cv_work, cv_done, cv_mem;
  std::deque<std::shared_ptr<Request>> queue;
  std::unordered_map<uint64_t, std::shared_ptr<Request>> reqs;
  std::vector<std::thread> workers;
  std::vector<hipStream_t> streams;
  static constexpr uint32_t kSmallWords = 512;  // a group's spans and the offsets of its texts
  struct Staging {
    uint8_t* buf[2] = {nullptr, nullptr};
    hipEvent_t ev[2] = {nullptr, nullptr};
    bool used[2] = {false, false};
    uint32_t next = 0;
    uint64_t* small = nullptr;  // pinned: kSmallWords values on their way to or from the device
    uint64_t* d_small = nullptr;  // device: the spans of a group
  };
  std::vector<Staging> staging;  // one per worker
  uint64_t next_id = 1;
  bool stop = false;
  std::atomic<uint64_t> launches{0};
};

namespace {

// ---- copies of many pieces by one launch ----------------------------------------------------
// A table's entries [0, n) on the way to a resident block: offsets rebased to the first word,
// counts, word bytes; or (off null) just bytes. Pieces are kernel arguments, kKeep at a time; a
// piece has a workgroup per kKeepSpan bytes: two copies of 8 bytes a thread, one after the other (32 KiB
// were sixteen: a table of 100 KiB took 7 us, now 3.6; 96 requests 1.58 -> 1.53 ms).
constexpr uint32_t kKeep = 32;
constexpr uint64_t kKeepSpan = 4096;
struct KeepItem {
  const uint64_t* off;
  const uint8_t* counts;
  const uint8_t* words;
  uint64_t n, count_bytes, word_bytes;  // count_bytes: of all entries
  uint64_t* d_off;
  uint8_t* d_counts;
  uint8_t* d_words;
};
struct KeepBatch {
  KeepItem item[kKeep];
  uint32_t first_block[kKeep];
  uint32_t n;
};

// bytes [a, b) of a copy of n bytes, eight at a time at any address
__device__ void copy_part(uint8_t* dst, const uint8_t* src, uint64_t n, uint64_t a, uint64_t b) {
  b = min(b, n);
  for (uint64_t i = a + threadIdx.x * 8; i < b; i += blockDim.x * 8) {
    if (i + 8 <= n) {
      uint64_t v;
      __builtin_memcpy(&v, src + i, 8);
      __builtin_memcpy(dst + i, &v, 8);
    } else {
      for (uint64_t q = i; q < n; ++q) dst[q] = src[q];
    }
  }
}

__global__ __launch_bounds__(256) void keep_kernel(KeepBatch K) {
  uint32_t x = 0;
  while (x + 1 < K.n && K.first_block[x + 1] <= blockIdx.x) ++x;
  const KeepItem& it = K.item[x];
  // the block's span of offsets | counts | words laid end to end (each rounded up to 8)
  const uint64_t a = (blockIdx.x - K.first_block[x]) * kKeepSpan, b = a + kKeepSpan;
  const uint64_t o = it.off ? (it.n + 1) * 8 : 0, c = (it.count_bytes + 7) & ~7ull;
  if (a < o) {
    const uint64_t base = it.off[0];
    for (uint64_t i = a / 8 + threadIdx.x; i < min(b, o) / 8; i += blockDim.x)
      it.d_off[i] = it.off[i] - base;
  }
  if (a < o + c && b > o)
    copy_part(it.d_counts, it.counts, it.count_bytes, a > o ? a - o : 0, b - o);
  if (b > o + c)
    copy_part(it.d_words, it.words + (it.off ? it.off[0] : 0), it.word_bytes,
              a > o + c ? a - o - c : 0, b - o - c);
}

hipError_t launch_keep(const std::vector<KeepItem>& items, hipStream_t s) {
  for (size_t i = 0; i < items.size();) {
    KeepBatch K;
    uint32_t blocks = 0;
    for (K.n = 0; i < items.size() && K.n < kKeep; ++i) {
      const KeepItem& it = items[i];
      const uint64_t bytes =
          (it.off ? (it.n + 1) * 8 : 0) + ((it.count_bytes + 7) & ~7ull) + it.word_bytes;
      if (!bytes) continue;
      K.item[K.n] = it;
      K.first_block[K.n++] = blocks;
      blocks += (uint32_t)((bytes + kKeepSpan - 1) / kKeepSpan);
    }
    if (!K.n) continue;
    hipLaunchKernelGGL(keep_kernel, dim3(blocks), dim3(256), 0, s, K);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Document d of a packed group (one workgroup each): its first entry, entries, word bytes and
// tokens (the sum of its counts), at out[4 d].
__global__ __launch_bounds__(256) void doc_span_kernel(wc_result t, uint64_t* out) {
  __shared__ unsigned long long s_sum;
  const uint64_t d = blockIdx.x, p = t.d_doc_ptr[d], n = t.d_doc_len[d];
  if (threadIdx.x == 0) s_sum = 0;
  __syncthreads();
  unsigned long long v = 0;
  for (uint64_t i = p + threadIdx.x; i < p + n; i += blockDim.x)
    v += t.count_bytes == 4 ? (unsigned long long)((const int32_t*)t.d_counts)[i]
                            : (unsigned long long)((const int64_t*)t.d_counts)[i];
  for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
  if ((threadIdx.x & 63) == 0 && v) atomicAdd(&s_sum, v);
  __syncthreads();
  if (threadIdx.x == 0) {
    out[4 * d] = p;
    out[4 * d + 1] = n;
    out[4 * d + 2] = n ? t.d_word_offsets[p + n] - t.d_word_offsets[p] : 0;
    out[4 * d + 3] = s_sum;
  }
}

uint64_t now_ns() {
  return (uint64_t)std::chrono::duration_cast<std::chrono::nanoseconds>(Clock::now().time_since_epoch()).count();
}

// Waits as the policy's answer says; false: the answer is final.
bool wait_memory(wc_server* S, std::unique_lock<std::mutex>& lk, wc::Admit a) {
  if (a == wc::Admit::kWait) S->cv_mem.wait(lk);
  else if (a == wc::Admit::kWaitRelease)
    S->cv_mem.wait_until(lk, Clock::time_point(std::chrono::nanoseconds(S->adm.deadline())));
  else return false;
  return true;
}

// A resident block for entries [e_begin, e_begin + n) of table t with nb word bytes: R's result
// points into it, and *item is the copy that fills it.
wc_status take_resident(wc_server* S, const wc_result& t, uint64_t e_begin, uint64_t n, uint64_t nb,
                        uint64_t tokens, Request* R, KeepItem* item, bool grace) {
  const uint32_t cb = t.count_bytes;
  const uint64_t bytes = (n + 1) * 8 + n * cb + nb + 64;
  uint8_t* mem = nullptr;
  {
    // This worker holds count memory; the policy (wc::Admission) lets it wait only while another
    // holder that is not itself waiting here, or the client, can still return memory.
    std::unique_lock<std::mutex> lk(S->mu);
    uint64_t off = 0;
    wc::Admit a;
    while ((a = S->adm.ask_resident(bytes, now_ns(), grace, &off)) != wc::Admit::kGranted && !S->stop) {
      ++S->adm.resident_waiters;
      const bool again = wait_memory(S, lk, a);
      --S->adm.resident_waiters;
      if (!again) break;
    }
    if (a != wc::Admit::kGranted) return WC_ENOMEM;
    mem = S->pool_mem + off;
  }
  uint64_t* d_off = (uint64_t*)mem;
  uint8_t* d_cnt = mem + (((n + 1) * 8 + 15) & ~15ull);
  uint8_t* d_words = d_cnt + ((n * cb + 15) & ~15ull);
  *item = KeepItem{t.d_word_offsets + e_begin, (const uint8_t*)t.d_counts + e_begin * cb, t.d_words,
                   n, n * cb, nb, d_off, d_cnt, d_words};
  R->resident = mem;
  memset(&R->res, 0, sizeof(R->res));
  R->res.n_entries = n;
  R->res.word_bytes = nb;
  R->res.count_bytes = cb;
  R->res.mode = WC_GLOBAL;
  R->res.n_docs = 1;
  R->res.total_tokens = tokens;
  R->res.d_word_offsets = d_off;
  R->res.d_words = d_words;
  R->res.d_counts = d_cnt;
  return WC_OK;
}

// The blocks taken are filled, and the requests of a failed copy give theirs back.
wc_status fill_residents(wc_server* S, const std::vector<KeepItem>& items, const std::vector<Request*>& rs,
                         hipStream_t s) {
  hipError_t e = launch_keep(items, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e == hipSuccess) return WC_OK;
  std::lock_guard<std::mutex> lk(S->mu);
  for (Request* R : rs) {
    S->adm.free_resident((uint64_t)(R->resident - S->pool_mem));
    R->resident = nullptr;
  }
  S->cv_mem.notify_all();
  return WC_EDEVICE;
}

// The whole table t into a resident block of R.
wc_status keep_table(wc_server* S, hipStream_t s, const wc_result& t, Request* R) {
  std::vector<KeepItem> item(1);
  const wc_status st = take_resident(S, t, 0, t.n_entries, t.word_bytes, t.total_tokens, R, &item[0], true);
  return st == WC_OK ? fill_residents(S, item, {R}, s) : st;
}

// Count memory for a request or a group (wc::Admission: in order, waiting while other requests, or
// with `grace` the client, can return memory); null when there is none.
uint8_t* pool_alloc_wait(wc_server* S, uint64_t bytes, bool grace) {
  std::unique_lock<std::mutex> lk(S->mu);
  uint64_t off = 0;
  wc::Admit a = wc::Admit::kFail;
  const uint64_t me = S->adm.arrive();
  while (!S->stop) {
    a = S->adm.ask_count(me, bytes, now_ns(), grace, &off);
    if (!wait_memory(S, lk, a)) break;
  }
  S->adm.leave(me);
  S->cv_mem.notify_all();
  return a == wc::Admit::kGranted ? S->pool_mem + off : nullptr;
}

void pool_free(wc_server* S, uint8_t* p) {
  std::lock_guard<std::mutex> lk(S->mu);
  S->adm.free_count((uint64_t)(p - S->pool_mem));
  S->cv_mem.notify_all();
}

// Free a resident table (under the lock).
void free_resident_locked(wc_server* S, Request* R) {
  if (R->resident) S->adm.free_resident((uint64_t)(R->resident - S->pool_mem));
  R->resident = nullptr;
  S->adm.progress(now_ns());
  S->cv_mem.notify_all();
}

// A merge is done with its inputs: a released input whose last reader this was is freed.
void unpin_inputs(wc_server* S, Request* M) {
  std::lock_guard<std::mutex> lk(S->mu);
  for (auto& in : M->merge_inputs)
    if (in->life.unpin()) free_resident_locked(S, in.get());
  M->merge_inputs.clear();
}

void finish(wc_server* S, Request* R, wc_status st) {
  std::lock_guard<std::mutex> lk(S->mu);
  R->status = st;
  R->state = 2;
  if (st == WC_OK) S->adm.progress(now_ns());
  R->t_done = now_s();
  R->text.clear();
  R->text.shrink_to_fit();
  S->cv_done.notify_all();
}

// Count a group of requests. One request: its own wc_count (its opts). Several small
// single-document requests: one per-document count, split per request.
// Host text to device memory through the worker's two pinned buffers, in order on stream s.
hipError_t upload(wc_server::Staging& W, uint8_t* dst, const uint8_t* src, uint64_t n,
                  hipStream_t s) {
  for (uint64_t off = 0; off < n; off += kStageBytes, W.next ^= 1) {
    const uint32_t k = W.next;  // alternates across calls too: small texts overlap as well
    const uint64_t m = std::min<uint64_t>(kStageBytes, n - off);
    if (W.used[k]) {
      hipError_t e = hipEventSynchronize(W.ev[k]);  // its previous transfer has finished
      if (e != hipSuccess) return e;
    }
    memcpy(W.buf[k], src + off, m);
    hipError_t e = hipMemcpyAsync(dst + off, W.buf[k], m, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipEventRecord(W.ev[k], s);
    if (e != hipSuccess) return e;
    W.used[k] = true;
  }
  return hipSuccess;
}

void run_group(wc_server* S, int idx, std::vector<std::shared_ptr<Request>>& G) {
  hipStream_t s = S->streams[idx];
  const double t0 = now_s();
  for (auto& r : G)
    if (!r->t_start) r->t_start = t0;
  if (G.size() == 1 && G[0]->merge) {
    Request* R = G[0].get();
    // The inputs were pinned when the merge was submitted (a release defers freeing their
    // resident tables until this merge is done); they were submitted before it, so they are
    // running or done: wait for them.
    std::vector<const wc_result*> ins;
    {
      std::unique_lock<std::mutex> lk(S->mu);
      for (auto& in : R->merge_inputs) {
        S->cv_done.wait(lk, [&] { return in->state == 2; });
        if (in->status != WC_OK) {
          ins.clear();
          break;
        }
        ins.push_back(&in->res);
      }
    }
    wc_status st = ins.empty() ? WC_EINVAL : WC_OK;
    wc_opts o = R->opts;
    wc_plan p;
    if (st == WC_OK) st = wc_merge_plan(ins.data(), (uint32_t)ins.size(), &o, &p);
    uint8_t* ws = nullptr;
    if (st == WC_OK && !(ws = pool_alloc_wait(S, p.workspace_bytes, true))) st = WC_ENOMEM;
    if (st == WC_OK) {
      wc_result t;
      st = wc_merge(ins.data(), (uint32_t)ins.size(), &o, ws, p.workspace_bytes, &t, s);
      S->launches++;
      if (st == WC_OK) st = keep_table(S, s, t, R);
    }
    if (ws) pool_free(S, ws);
    unpin_inputs(S, R);  // the merge's stream is synchronised: nothing reads the inputs now
    return finish(S, R, st);
  }
  // the texts on the device: one buffer for the group (a device text counted alone stays where it is)
  uint64_t total = 0;
  for (auto& r : G) total += r->len;
  const bool packed = G.size() > 1;
  const bool in_place = !packed && G[0]->dev_text;
  uint64_t n_docs_all = 0;
  for (auto& r : G) n_docs_all += packed ? 1 : r->offsets.size() - 1;
  wc_opts o = G[0]->opts;
  wc_server::Staging& W = S->staging[idx];
  if (packed) {
    o.mode = WC_PER_DOC;
    o.tuning = nullptr;
    o.table_slots = 0;
    o.word_bytes_cap = total;  // room for any texts (the group is small): counted once
    o.debug_flags = (o.debug_flags & ~WC_DEBUG_DIRECT) | WC_DEBUG_DOCS;
  }
  wc_status st = WC_OK;
  for (int attempt = 0; attempt < 8; ++attempt) {
    wc_plan p;
    st = wc_count_plan(total, n_docs_all, &o, &p);
    if (st != WC_OK) break;
    if (packed && p.workspace_bytes > S->budget / 4 && o.word_bytes_cap == total) {
      o.word_bytes_cap = 0;  // a tight budget: the default room
      st = wc_count_plan(total, n_docs_all, &o, &p);
      if (st != WC_OK) break;
    }
    const uint64_t off_bytes = (n_docs_all + 1) * 8;
    const uint64_t text_bytes = in_place ? 0 : (total + 255) & ~255ull;
    const uint64_t need = p.workspace_bytes + text_bytes + off_bytes + 512;
    if (need > S->budget) {
      st = WC_ENOMEM;
      break;
    }
    uint8_t* mem = pool_alloc_wait(S, need, !packed);
    if (!mem) {
      st = WC_ENOMEM;
      break;
    }
    uint8_t* buf = mem;
    const uint8_t* d_text = in_place ? G[0]->dev_text : buf;
    uint64_t* d_off = (uint64_t*)(mem + text_bytes);
    uint8_t* ws = (uint8_t*)d_off + ((off_bytes + 255) & ~255ull);
    std::vector<uint64_t> off;
    off.reserve(n_docs_all + 1);
    uint64_t pos = 0;
    hipError_t e = hipSuccess;
    std::vector<KeepItem> gather;  // device texts of a group
    for (auto& r : G) {
      if (in_place) {
      } else if (r->dev_text) {
        if (packed) gather.push_back(KeepItem{nullptr, nullptr, r->dev_text, 0, 0, r->len, nullptr, nullptr, buf + pos});
        else e = hipMemcpyAsync(buf + pos, r->dev_text, r->len, hipMemcpyDeviceToDevice, s);
      } else if (r->host_text && r->len) {  // in place: pinned memory goes straight to the DMA engine
        e = hipMemcpyAsync(buf + pos, r->host_text, r->len, hipMemcpyHostToDevice, s);
      } else if (r->len) {
        e = upload(W, buf + pos, r->text.data(), r->len, s);
      }
      if (e != hipSuccess) break;
      if (packed) {
        off.push_back(pos);
      } else {
        for (size_t i = 0; i + 1 < r->offsets.size(); ++i) off.push_back(r->offsets[i]);
      }
      pos += r->len;
    }
    if (packed) off.push_back(pos);
    else off.push_back(G[0]->offsets.back());
    if (e == hipSuccess) e = launch_keep(gather, s);
    if (e == hipSuccess) {
      // (few offsets go through the worker's pinned words; the call waits before their next use)
      const uint64_t* from = off.data();
      if (off.size() <= wc_server::kSmallWords) {
        memcpy(W.small, off.data(), off_bytes);
        from = W.small;
      }
      e = hipMemcpyAsync(d_off, from, off_bytes, hipMemcpyHostToDevice, s);
    }
    if (e != hipSuccess) {
      pool_free(S, mem);
      st = WC_EDEVICE;
      break;
    }
    wc_result t;
    st = wc_count(d_text, total, d_off, n_docs_all, &o, ws, p.workspace_bytes, &t, s);
    S->launches++;
    if (st == WC_ETABLEFULL) {  // a global or (document, word) table: twice the slots
      o.table_slots = 2 * p.table_slots;
      pool_free(S, mem);
      continue;
    }
    if (st == WC_ENOMEM && !(t.word_bytes <= p.word_bytes_cap && t.table_slots <= p.table_slots)) {
      o.word_bytes_cap = std::max<uint64_t>(t.word_bytes, 3 * t.n_entries) * 5 / 4 + 4096;
      if (o.mode == WC_PER_DOC && t.table_slots > p.table_slots) {
        uint64_t want = 1;
        while (want < 2 * t.table_slots) want <<= 1;
        o.table_slots = want;
      }
      pool_free(S, mem);
      continue;
    }
    if (st == WC_OK) {
      if (!packed) {
        st = keep_table(S, s, t, G[0].get());
      } else {
        hipLaunchKernelGGL(doc_span_kernel, dim3((uint32_t)G.size()), dim3(256), 0, s, t, W.d_small);
        e = hipGetLastError();
        if (e == hipSuccess)
          e = hipMemcpyAsync(W.small, W.d_small, G.size() * 32, hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e != hipSuccess) st = WC_EDEVICE;
        std::vector<KeepItem> items;
        std::vector<Request*> taken;
        for (size_t i = 0; st == WC_OK && i < G.size(); ++i) {
          const uint64_t* v = W.small + 4 * i;
          KeepItem item;
          st = take_resident(S, t, v[0], v[1], v[2], v[3], G[i].get(), &item, false);
          if (st == WC_OK) {
            items.push_back(item);
            taken.push_back(G[i].get());
          }
        }
        const wc_status filled = fill_residents(S, items, taken, s);
        if (filled != WC_OK) st = filled;
      }
    }
    pool_free(S, mem);
    break;
  }
  if (packed && st == WC_ENOMEM) {
    // Too little memory for the group, which each of its requests may have enough of: those without
    // a table yet are counted one by one. (The group's count takes at least 8 MiB, for words that do
    // not fit LDS; a request of 32 KiB alone less than 1.)
    for (auto& r : G) {
      if (r->resident) {
        finish(S, r.get(), WC_OK);
      } else {
        std::vector<std::shared_ptr<Request>> one{r};
        run_group(S, idx, one);
      }
    }
    return;
  }
  for (auto& r : G) finish(S, r.get(), st);
}

void release_staging(wc_server* S) {
  for (auto& W : S->staging) {
    for (int k = 0; k < 2; ++k) {
      if (W.ev[k]) (void)hipEventSynchronize(W.ev[k]);
      if (W.ev[k]) (void)hipEventDestroy(W.ev[k]);
      if (W.buf[k]) (void)hipHostFree(W.buf[k]);
      W.ev[k] = nullptr;
      W.buf[k] = nullptr;
    }
    if (W.small) (void)hipHostFree(W.small);
    if (W.d_small) (void)hipFree(W.d_small);
    W.small = nullptr;
    W.d_small = nullptr;
  }
}

void worker(wc_server* S, int idx) {
  hipSetDevice(S->device);
  while (true) {
    std::vector<std::shared_ptr<Request>> G;
    {
      std::unique_lock<std::mutex> lk(S->mu);
      S->cv_work.wait(lk, [&] { return S->stop || !S->queue.empty(); });
      if (S->stop && S->queue.empty()) return;
      auto first = S->queue.front();
      S->queue.pop_front();
      first->state = 1;
      G.push_back(first);
      auto small = [](const Request& r) {
        return !r.merge && r.offsets.size() == 2 && r.offsets[0] == 0 && r.offsets[1] == r.len &&
               r.len <= kSmallBytes;
      };
      if (small(*first)) {
        while (!S->queue.empty() && G.size() < kPackDocs) {
          auto& nx = S->queue.front();
          if (!small(*nx) || nx->opts.count_bytes != first->opts.count_bytes ||
              nx->opts.tokenizer != first->opts.tokenizer ||
              nx->opts.debug_hash_bits != first->opts.debug_hash_bits)
            break;
          nx->state = 1;
          G.push_back(nx);
          S->queue.pop_front();
        }
      }
    }
    run_group(S, idx, G);
  }
}

}  // namespace

extern "C" {

wc_status wc_server_create(int device, uint64_t mem_budget, uint32_t max_streams,
                           wc_server** out) {
  if (!out || mem_budget < (1ull << 20) || max_streams == 0 || max_streams > 16) return WC_EINVAL;
  if (hipSetDevice(device) != hipSuccess) return WC_EDEVICE;
  wc_server* S = new wc_server();
  S->device = device;
  S->budget = mem_budget;
  if (hipMalloc((void**)&S->pool_mem, mem_budget) != hipSuccess) {
    delete S;
    return WC_ENOMEM;
  }
  S->adm.init(mem_budget);
  for (uint32_t i = 0; i < max_streams; ++i) {
    hipStream_t s;
    if (hipStreamCreateWithFlags(&s, hipStreamNonBlocking) != hipSuccess) {
      for (auto x : S->streams) hipStreamDestroy(x);
      hipFree(S->pool_mem);
      delete S;
      return WC_EDEVICE;
    }
    S->streams.push_back(s);
  }
  S->staging.resize(max_streams);
  for (auto& W : S->staging) {
    for (int k = 0; k < 2; ++k) {
      if (hipHostMalloc((void**)&W.buf[k], kStageBytes, hipHostMallocDefault) != hipSuccess ||
          hipEventCreateWithFlags(&W.ev[k], hipEventDisableTiming) != hipSuccess ||
          (k == 0 && (hipHostMalloc((void**)&W.small, wc_server::kSmallWords * 8, hipHostMallocDefault) !=
                          hipSuccess ||
                      hipMalloc((void**)&W.d_small, kPackDocs * 32) != hipSuccess))) {
        release_staging(S);
        for (auto x : S->streams) hipStreamDestroy(x);
        hipFree(S->pool_mem);
        delete S;
        return WC_EDEVICE;
      }
    }
  }
  for (uint32_t i = 0; i < max_streams; ++i) S->workers.emplace_back(worker, S, (int)i);
  *out = S;
  return WC_OK;
}

wc_status wc_server_submit(wc_server* S, const uint8_t* text, uint64_t len,
                           const uint64_t* offsets, uint64_t n_docs, int text_on_device,
                           const wc_opts* opts, uint64_t* req_id) {
  if (!S || !req_id || !opts || (len && !text) || !offsets) return WC_EINVAL;
  if (text_on_device != WC_TEXT_HOST_COPY && text_on_device != WC_TEXT_DEVICE &&
      text_on_device != WC_TEXT_HOST_IN_PLACE)
    return WC_EINVAL;
  if (opts->count_bytes != 4 && opts->count_bytes != 8) return WC_EINVAL;
  if (opts->mode != WC_GLOBAL) return WC_EINVAL;  // per-request tables are global tables
  for (uint64_t i = 0; i < n_docs; ++i)
    if (offsets[i] > offsets[i + 1]) return WC_EINVAL;
  if (offsets[n_docs] > len) return WC_EINVAL;
  // admission test: the request must fit the budget on its own
  wc_plan p;
  wc_opts o = *opts;
  o.tuning = nullptr;
  wc_status st = wc_count_plan(len, n_docs, &o, &p);
  if (st != WC_OK) return st;
  auto fits = [&] { return p.workspace_bytes + len + (n_docs + 1) * 8 + 1024 <= S->budget; };
  if (!fits() && len < (256ull << 20)) {
    // below the two-pass size the one-pass kernel needs less memory than the partitioned ones
    o.debug_flags |= WC_DEBUG_DIRECT;
    if ((st = wc_count_plan(len, n_docs, &o, &p)) != WC_OK) return st;
  }
  if (!fits()) return WC_ENOMEM;
  auto R = std::make_shared<Request>();
  R->len = len;
  if (text_on_device == WC_TEXT_DEVICE) R->dev_text = text;
  else if (text_on_device == WC_TEXT_HOST_IN_PLACE) R->host_text = text;
  else R->text.assign(text, text + len);
  R->offsets.assign(offsets, offsets + n_docs + 1);
  R->opts = o;
  R->t_submit = now_s();
  {
    std::lock_guard<std::mutex> lk(S->mu);
    R->id = S->next_id++;
    S->reqs[R->id] = R;
    S->queue.push_back(R);
    *req_id = R->id;
  }
  S->cv_work.notify_one();
  return WC_OK;
}

wc_status wc_server_poll(wc_server* S, uint64_t id, wc_result* out) {
  if (!S || !out) return WC_EINVAL;
  std::lock_guard<std::mutex> lk(S->mu);
  auto it = S->reqs.find(id);
  if (it == S->reqs.end()) return WC_EINVAL;
  if (it->second->state != 2) return WC_EAGAIN;
  *out = it->second->res;
  return it->second->status;
}

wc_status wc_server_wait(wc_server* S, uint64_t id, wc_result* out) {
  if (!S || !out) return WC_EINVAL;
  std::unique_lock<std::mutex> lk(S->mu);
  auto it = S->reqs.find(id);
  if (it == S->reqs.end()) return WC_EINVAL;
  auto R = it->second;
  S->cv_done.wait(lk, [&] { return R->state == 2; });
  *out = R->res;
  return R->status;
}

wc_status wc_server_times(wc_server* S, uint64_t id, double* submit_s, double* start_s,
                          double* done_s) {
  if (!S) return WC_EINVAL;
  std::lock_guard<std::mutex> lk(S->mu);
  auto it = S->reqs.find(id);
  if (it == S->reqs.end()) return WC_EINVAL;
  if (submit_s) *submit_s = it->second->t_submit;
  if (start_s) *start_s = it->second->t_start;
  if (done_s) *done_s = it->second->t_done;
  return it->second->state == 2 ? WC_OK : WC_EAGAIN;
}

wc_status wc_server_merge(wc_server* S, const uint64_t* ids, uint32_t k, const wc_opts* opts,
                          uint64_t* new_id) {
  if (!S || !new_id || !ids || k == 0) return WC_EINVAL;
  if (opts && opts->count_bytes != 4 && opts->count_bytes != 8) return WC_EINVAL;
  auto R = std::make_shared<Request>();
  R->merge = true;
  R->merge_ids.assign(ids, ids + k);
  wc_opts o{};
  o.count_bytes = opts ? opts->count_bytes : 8;
  R->opts = o;
  R->t_submit = now_s();
  {
    std::lock_guard<std::mutex> lk(S->mu);
    // pin the inputs now: releasing one before the merge has read it defers the free
    for (uint32_t i = 0; i < k; ++i) {
      auto it = S->reqs.find(ids[i]);
      if (it == S->reqs.end()) return WC_EINVAL;  // nothing pinned yet
      R->merge_inputs.push_back(it->second);
    }
    for (auto& in : R->merge_inputs) in->life.pin();
    R->id = S->next_id++;
    S->reqs[R->id] = R;
    S->queue.push_back(R);
    *new_id = R->id;
  }
  S->cv_work.notify_one();
  return WC_OK;
}

wc_status wc_server_release(wc_server* S, uint64_t id) {
  if (!S) return WC_EINVAL;
  std::shared_ptr<Request> R;
  {
    std::unique_lock<std::mutex> lk(S->mu);
    auto it = S->reqs.find(id);
    if (it == S->reqs.end()) return WC_EINVAL;
    R = it->second;
    S->cv_done.wait(lk, [&] { return R->state == 2; });
    auto again = S->reqs.find(id);  // the wait may have let another thread in
    if (again == S->reqs.end() || again->second != R) return WC_EINVAL;
    S->reqs.erase(again);
    // a merge that will read the table frees it when done (ResidentLife)
    if (R->life.release()) free_resident_locked(S, R.get());
  }
  return WC_OK;
}

uint64_t wc_server_launches(wc_server* S) { return S ? S->launches.load() : 0; }

wc_status wc_server_destroy(wc_server* S) {
  if (!S) return WC_OK;
  {
    std::lock_guard<std::mutex> lk(S->mu);
    S->stop = true;
  }
  S->cv_work.notify_all();
  S->cv_mem.notify_all();
  for (auto& t : S->workers) t.join();
  release_staging(S);
  for (auto s : S->streams) hipStreamDestroy(s);
  hipFree(S->pool_mem);
  delete S;
  return WC_OK;
}

}  // extern "C"
