// How muon_adamw_step cuts its list into launches: plain C++, no HIP include, so that the tests build it with the host
// compiler alone.
#pragma once
#include <algorithm>
#include <cstdint>

#include "../../include/muon.h"
#include "muon_tables.h"

namespace muon {

constexpr int kAdamwSlots = 64;                  // tensors (or pieces of one) per launch: 3.3 KB of kernel arguments
static_assert((kAdamwSlots & (kAdamwSlots - 1)) == 0, "the kernel finds a block's tensor by halving steps");
constexpr int kAdamwSpan = 1024;                 // elements per block of 256 threads
// A launch holds less than 2^32 work-items: 17.2 G elements, 206 GB of bf16 parameters, gradients and fp32 moments, which
// fits the device's memory.  Longer lists and larger tensors go on in the next launch.
constexpr int64_t kAdamwMaxBlocks = (int64_t{1} << 24) - 1;
constexpr int64_t kAdamwMaxNumel = int64_t{1} << 42;           // per tensor

// Travels by value in the kernel arguments.
struct AdamwBatch {
  void* p[kAdamwSlots];
  const void* g[kAdamwSlots];
  float* m[kAdamwSlots];
  float* v[kAdamwSlots];
  long long numel[kAdamwSlots];
  int block_start[kAdamwSlots + 1];   // first block of each tensor; [n] = total blocks
  int p_dtype[kAdamwSlots], g_dtype[kAdamwSlots];
  int n;
};

// Position in the list: tensors before `tensor` and the first `element` elements of that one are in earlier launches.
struct AdamwCursor {
  int32_t tensor = 0;
  int64_t element = 0;                // a multiple of kAdamwSpan
};

// Fills `b` with the next launch's pieces and moves the cursor behind them.  Returns the launch's blocks (0: list done).
inline int adamw_next_batch(const muon_adamw_param* params, int32_t n, AdamwCursor& at, AdamwBatch& b) {
  int64_t blocks = 0;
  b.n = 0;
  while (at.tensor < n && b.n < kAdamwSlots && blocks < kAdamwMaxBlocks) {
    const muon_adamw_param& q = params[at.tensor];
    const int64_t e = at.element, most = (kAdamwMaxBlocks - blocks) * kAdamwSpan, len = std::min<int64_t>(q.numel - e, most);
    const int k = b.n++;
    b.p[k] = static_cast<char*>(q.p) + e * (q.p_dtype == kDtypeBF16 ? 2 : 4);
    b.g[k] = static_cast<const char*>(q.g) + e * (q.g_dtype == kDtypeBF16 ? 2 : 4);
    b.m[k] = q.m + e;
    b.v[k] = q.v + e;
    b.numel[k] = len;
    b.p_dtype[k] = q.p_dtype;
    b.g_dtype[k] = q.g_dtype;
    b.block_start[k] = (int)blocks;
    blocks += (len + kAdamwSpan - 1) / kAdamwSpan;
    if (e + len == q.numel) {
      ++at.tensor;
      at.element = 0;
    } else {
      at.element = e + len;
    }
  }
  b.block_start[b.n] = (int)blocks;
  return (int)blocks;
}

}  // namespace muon
