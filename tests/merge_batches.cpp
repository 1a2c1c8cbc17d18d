// Host test of the launches that a merge's inputs are cut into (for_merge_batches of
// paper_2206_05269_amd/csrc/wc_internal.h): every input is in one launch, in order, the workgroups of
// a launch are those of its inputs, and no launch that holds several inputs has 2^32 threads or
// more. No GPU. Exit status 0 when every check holds.
#include <stdio.h>

#include <vector>

#include "wc_internal.h"

static int failures = 0;
#define CHECK(c)                                                      \
  do {                                                                \
    if (!(c)) {                                                       \
      printf("FAIL %s:%d: %s\n", __FILE__, __LINE__, #c);             \
      ++failures;                                                     \
    }                                                                 \
  } while (0)

static void run(const std::vector<uint64_t>& sizes, uint32_t span) {
  std::vector<wc::MergeInput> in(sizes.size());
  for (size_t i = 0; i < in.size(); ++i) {
    in[i].n = sizes[i];
    in[i].column = (uint32_t)i;
  }
  std::vector<uint32_t> seen;
  CHECK(wc::for_merge_batches(in.data(), (uint32_t)in.size(), span,
                              [&](const wc::MergeBatch& M, uint32_t blocks) {
                                CHECK(M.n >= 1 && M.n <= wc::kMergeInputs);
                                uint64_t at = 0;
                                for (uint32_t i = 0; i < M.n; ++i) {
                                  CHECK(M.first_block[i] == at);
                                  at += (M.in[i].n + span - 1) / span;
                                  seen.push_back(M.in[i].column);
                                }
                                CHECK(at == blocks);
                                CHECK(M.n == 1 || (uint64_t)blocks * 1024 < (1ull << 32));
                                return hipSuccess;
                              }) == hipSuccess);
  std::vector<uint32_t> want;
  for (size_t i = 0; i < sizes.size(); ++i)
    if (sizes[i]) want.push_back((uint32_t)i);
  CHECK(seen == want);
}

int main() {
  for (uint32_t span : {256u, 4096u}) {
    run({}, span);
    run({0, 0}, span);
    run({1, 0, 255, 256, 257, 4095, 4096, 4097}, span);
    run(std::vector<uint64_t>(100, 1000), span);
    run(std::vector<uint64_t>(7, 3000000000ull), span);
    run({5, 4000000000ull, 1000000000ull, 0, 70000000ull, 900000000ull, 1}, span);
  }
  if (!failures) printf("all ok\n");
  return failures ? 1 : 0;
}
