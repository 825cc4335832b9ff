// Checks how muon_adamw_step cuts a list into launches (built by tests/test_adamw_batches.py with the host compiler alone):
// every launch stays below 2^32 work-items of 256-thread blocks, and the launches together take every element of every
// tensor once, in order, at the right addresses.  No address is followed.
#include <cstdio>
#include <cstring>
#include <vector>

#include "../paper_2502_16982_amd/csrc/adamw_batch.h"

using namespace muon;

static int failures = 0;
#define CHECK(cond)                                                                                    \
  do {                                                                                                 \
    if (!(cond)) {                                                                                     \
      std::fprintf(stderr, "list %d, launch %d: CHECK failed: %s\n", list_no, launches, #cond);        \
      ++failures;                                                                                      \
    }                                                                                                  \
  } while (0)

static int list_no = 0;

static void walk(const std::vector<int64_t>& sizes, int64_t want_launches) {
  int launches = 0;
  std::vector<muon_adamw_param> list(sizes.size());
  uintptr_t next = uintptr_t{1} << 50;
  for (size_t i = 0; i < sizes.size(); ++i) {
    muon_adamw_param& q = list[i];
    q.numel = sizes[i];
    q.p_dtype = i % 2 ? MUON_F32 : MUON_BF16;
    q.g_dtype = i % 3 ? MUON_BF16 : MUON_F32;
    q.p = reinterpret_cast<void*>(next);
    q.g = reinterpret_cast<void*>(next += 4 * (uintptr_t)sizes[i] + 6);
    q.m = reinterpret_cast<float*>(next += 4 * (uintptr_t)sizes[i] + 4);
    q.v = reinterpret_cast<float*>(next += 4 * (uintptr_t)sizes[i] + 4);
    next += 4 * (uintptr_t)sizes[i] + 8;
  }
  AdamwCursor at;
  AdamwBatch b;
  size_t tensor = 0;
  int64_t done = 0;                   // elements of list[tensor] in earlier pieces
  while (const int blocks = adamw_next_batch(list.data(), (int32_t)list.size(), at, b)) {
    ++launches;
    CHECK(blocks > 0 && (uint64_t)blocks * 256 < (uint64_t{1} << 32));
    CHECK(b.n >= 1 && b.n <= kAdamwSlots && b.block_start[0] == 0 && b.block_start[b.n] == blocks);
    for (int k = 0; k < b.n; ++k) {
      CHECK(tensor < list.size());
      if (tensor >= list.size()) return;
      const muon_adamw_param& q = list[tensor];
      CHECK(b.numel[k] >= 1 && done + b.numel[k] <= q.numel && done % kAdamwSpan == 0);
      CHECK(b.block_start[k + 1] - b.block_start[k] == (b.numel[k] + kAdamwSpan - 1) / kAdamwSpan);
      CHECK(b.p_dtype[k] == q.p_dtype && b.g_dtype[k] == q.g_dtype);
      CHECK((char*)b.p[k] == (char*)q.p + done * (q.p_dtype == MUON_BF16 ? 2 : 4));
      CHECK((const char*)b.g[k] == (const char*)q.g + done * (q.g_dtype == MUON_BF16 ? 2 : 4));
      CHECK(b.m[k] == q.m + done && b.v[k] == q.v + done);
      done += b.numel[k];
      if (done == q.numel) {
        ++tensor;
        done = 0;
      }
    }
    if (launches > 1000) return;
  }
  CHECK(tensor == list.size() && done == 0);
  CHECK(launches == want_launches);
  ++list_no;
}

int main() {
  const int64_t full = kAdamwMaxBlocks * kAdamwSpan;           // elements one launch can take
  walk({1}, 1);
  walk({1, 1023, 1024, 1025, 4099}, 1);
  walk(std::vector<int64_t>(64, 2048), 1);
  walk(std::vector<int64_t>(65, 2048), 2);
  walk(std::vector<int64_t>(130, 3), 3);
  walk({full}, 1);
  walk({full + 1}, 2);
  walk({full - 1024, 1024, 5}, 2);                             // the list's end meets the launch's
  walk({full - 1023, 2000}, 2);
  walk({int64_t{1} << 34}, 2);                                 // 206 GB of bf16 p, g and fp32 m, v
  walk(std::vector<int64_t>(64, 300000007), 2);                // 19.2 G elements
  walk({7, 3 * full + 9, 7}, 4);
  walk({kAdamwMaxNumel}, 257);
  if (failures) {
    std::fprintf(stderr, "%d checks failed\n", failures);
    return 1;
  }
  std::printf("batches ok: %d lists\n", list_no);
  return 0;
}
