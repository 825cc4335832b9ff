// Newton-Schulz products of lists with matrices iterated on their Gram matrix (the planner's gram_route).  A launch takes two
// sides: the next product of the matrices iterated as Eq. 2 is written, and the next product of the others; either may be empty.
// A side has its own tables, coefficients and types: operands bf16 or f16, the L operand contiguous along k or K-major; symmetric
// products write the type they read, apply products bf16 or f16.  The tiles, their pipelines and what bounds them are those of
// kernels_gemm_bf16.hip, gemm_tile64.h and gemm_ring128.h; what is new is that
// two sides share a launch, since each alone leaves compute units idle in its last round and one chain of launches is shorter than
// two.  us per step, all matrices as Eq. 2 / this: 4 of 1024^2 with 3 of 1024 x 4096 (fine launches) 472 / 453, twelve of those (coarse
// ones) 4622 / 4276, 4 of 4096^2 with 3 of 4096 x 11008 12992 / 11960.
// Fine launches pair anything with anything: blocks below blocks_x are the first side's.  In coarse launches the symmetric
// products share a kernel, from one table that is dealt as one (side by side, each dealt by itself, 30 of 1024^2 with 3 of 1024 x 4096
// took 82 us per polynomial launch, from one table 70, where all of them as Eq. 2 take 69): a kernel with the K-major bodies too
// spilled more and took a third longer on every product.  An apply product in coarse tiles takes in a product that is all 128-wide blocks
// (ns_pair_beside_kernel; one tile per block: 5 to 9 registers are spilled, none in a K loop), and the other side's apply product where one table of both
// saves a round (ns_pair_apply_kernel).
#include "gemm_tile256.h"
#include "gemm_planes.h"
#include "gemm_tile64.h"
#include "gemm_ring128.h"

namespace muon {
namespace {

constexpr size_t kLds128 = TileCfg<128, 128>::lds_bytes(2);
constexpr size_t kLds256 = TileCfg<256, 256>::lds_bytes(2);
constexpr size_t kLds512 = TileCfg<512, 128>::lds_bytes(2);

// The side of block `b`, chosen field by field (an indexed copy of the arguments would live in scratch memory).
__device__ __forceinline__ GemmSide pick_side(const GemmSide& x, const GemmSide& y, bool first) {
  GemmSide s;
  s.probs = first ? x.probs : y.probs;
  s.tiles = first ? x.tiles : y.tiles;
  s.n_tiles = first ? x.n_tiles : y.n_tiles;
  s.beta_acc = first ? x.beta_acc : y.beta_acc;
  s.beta_e = first ? x.beta_e : y.beta_e;
  s.diag_add = first ? x.diag_add : y.diag_add;
  s.alpha_idx = first ? x.alpha_idx : y.alpha_idx;
  s.kind = first ? x.kind : y.kind;
  s.gain = first ? x.gain : y.gain;
  return s;
}

// f(LKM, IN{}, OUT{}) for a side's operand layout and types
template <typename F>
__device__ __forceinline__ void with_operands(int kind, F&& f) {
  if (kind & kSideKMajor) {
    if (kind & kSideInF16) f(std::true_type{}, F16{}, Any16{});
    else f(std::true_type{}, Bf16{}, Any16{});
  } else {
    if (kind & kSideInF16) f(std::false_type{}, F16{}, F16{});
    else f(std::false_type{}, Bf16{}, Bf16{});
  }
}

__global__ __launch_bounds__(256, 2) void ns_pair_fine_kernel(GemmSide x, GemmSide y, int blocks_x) {
  extern __shared__ __align__(16) unsigned char smem[];
  const bool first = (int)blockIdx.x < blocks_x;
  const GemmSide s = pick_side(x, y, first);
  const int t = first ? (int)blockIdx.x : (int)blockIdx.x - blocks_x;
  if (t >= s.n_tiles) return;
  const GemmTile tile = load_tile(s.tiles, t);
  const GemmProblem p = s.probs[tile.prob];
  with_operands(s.kind, [&](auto lkm, auto in, auto out) {
    gemm_tile_body<128, 128, 2, 2, 2, decltype(lkm)::value, decltype(in), decltype(out)>(p, tile, smem, s.beta_acc, s.beta_e, s.alpha_idx, s.diag_add,
                                                                                __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), (s.kind & kSideOutF16) != 0);
  });
}

// One block of a compute unit per entry: as ns_ring128_bf16_kernel.
__global__ __launch_bounds__(256, 1) void ns_pair_ring128_kernel(GemmSide x, GemmSide y, int blocks_x, double eps) {
  extern __shared__ __align__(16) unsigned char smem[];
  const bool first = (int)blockIdx.x < blocks_x;
  const GemmSide s = pick_side(x, y, first);
  const int t = first ? (int)blockIdx.x : (int)blockIdx.x - blocks_x;
  if (t >= s.n_tiles) return;
  const GemmTile tile = load_tile(s.tiles, t);
  const GemmProblem p = s.probs[tile.prob];
  with_operands(s.kind, [&](auto lkm, auto in, auto out) {
    gemm_ring128_body<decltype(lkm)::value, decltype(in), decltype(out)>(p, tile.r0 * kTileUnit, tile.c0 * kTileUnit, (tile.flags & kTileDiagonal) != 0, smem,
                                                                s.beta_acc, s.beta_e, s.alpha_idx, eps, s.diag_add, (s.kind & kSideOutF16) != 0, s.gain);
  });
}

// Entry and quarter of a block: as in ns_tile64_gemm_bf16_kernel.
template <int NST, int BLOCKS>
__global__ __launch_bounds__(256, BLOCKS) void ns_pair_tile64_kernel(GemmSide x, GemmSide y, int blocks_x, double eps) {
  extern __shared__ __align__(16) unsigned char smem[];
  const bool first = (int)blockIdx.x < blocks_x;
  const GemmSide s = pick_side(x, y, first);
  const int b = first ? (int)blockIdx.x : (int)blockIdx.x - blocks_x;
  const int t = (b >> 5) * 8 + (b & 7), quarter = (b >> 3) & 3;
  if (t >= s.n_tiles) return;
  const GemmTile tile = load_tile(s.tiles, t);
  const bool on_diag = (tile.flags & kTileDiagonal) != 0;
  if (on_diag && quarter == 2) return;           // below the diagonal: the mirror image of quarter 1
  const GemmProblem p = s.probs[tile.prob];
  const int row0 = tile.r0 * kTileUnit + 64 * (quarter >> 1), col0 = tile.c0 * kTileUnit + 64 * (quarter & 1);
  with_operands(s.kind, [&](auto lkm, auto in, auto out) {
    gemm_tile64_body<decltype(lkm)::value, 4, NST, decltype(in), decltype(out)>(p, row0, col0, on_diag && quarter != 1, smem, s.beta_acc, s.beta_e,
                                                                       s.alpha_idx, eps, s.diag_add, (s.kind & kSideOutF16) != 0, s.gain);
  });
}

// Entry and sixteenth of a block: as in ns_tile32_gemm_bf16_kernel.
__global__ __launch_bounds__(64) void ns_pair_tile32_kernel(GemmSide x, GemmSide y, int blocks_x, double eps) {
  extern __shared__ __align__(16) unsigned char smem[];
  const bool first = (int)blockIdx.x < blocks_x;
  const GemmSide s = pick_side(x, y, first);
  const int b = first ? (int)blockIdx.x : (int)blockIdx.x - blocks_x;
  const int t = (b >> 7) * 8 + (b & 7), part = (b >> 3) & 15;
  if (t >= s.n_tiles) return;
  const GemmTile tile = load_tile(s.tiles, t);
  const bool on_diag = (tile.flags & kTileDiagonal) != 0;
  if (on_diag && (part >> 2) > (part & 3)) return;   // below the diagonal: a mirror image
  const GemmProblem p = s.probs[tile.prob];
  with_operands(s.kind, [&](auto lkm, auto in, auto out) {
    gemm_tile64_body<decltype(lkm)::value, 1, kRing32, decltype(in), decltype(out)>(p, tile.r0 * kTileUnit + 32 * (part >> 2), tile.c0 * kTileUnit + 32 * (part & 3),
                                                                           on_diag && (part >> 2) == (part & 3), smem, s.beta_acc, s.beta_e,
                                                                           s.alpha_idx, eps, s.diag_add, (s.kind & kSideOutF16) != 0, s.gain);
  });
}

// One side with f16 among its types, one block per entry or, persistent, per compute unit: as in ns_gemm_bf16_kernel.  (Coarse bodies take the
// type of their results at run time even where there is one: with it known, 61 registers instead of 29 were spilled in the shared kernel
// below, 25 instead of 2 and 8 instead of none here.)
template <bool LKM, typename IN>
__global__ __launch_bounds__(256, 1) void ns_pair_coarse_kernel(const GemmProblem* __restrict__ probs, const GemmTile* __restrict__ tiles, int n_tiles,
                                                                float beta_acc, float beta_e, int alpha_idx, float diag_add, int out_f16) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int wave_id = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int t = blockIdx.x; t < n_tiles; t += gridDim.x) {
    const GemmTile tile = load_tile(tiles, t);
    const GemmProblem p = probs[tile.prob];
    const int shape = __builtin_amdgcn_readfirstlane(tile.shape);
    if (shape == kShape512x128) {
      gemm_tile_body<512, 128, 4, 1, 2, LKM, IN, Any16>(p, tile, smem, beta_acc, beta_e, alpha_idx, diag_add, wave_id, out_f16 != 0);
    } else if (!LKM && shape == kShape256Diag) {
      if constexpr (!LKM) diag_tile_body<IN>(p, tile, smem, beta_acc, beta_e, alpha_idx, diag_add, wave_id);
    } else {
      gemm_tile_body<256, 256, 2, 2, 2, LKM, IN, Any16>(p, tile, smem, beta_acc, beta_e, alpha_idx, diag_add, wave_id, out_f16 != 0);
    }
    __syncthreads();        // every wave has read its part of the LDS images: the next tile may overwrite them
  }
}

// Symmetric products of both sides from one table (kTileSecond marks the second's tiles).
template <typename IN>
__device__ __forceinline__ void coarse_sym_tile(const GemmSide& s, const GemmTile& tile, unsigned char* smem, int wave_id) {
  const GemmProblem p = s.probs[tile.prob];
  const int shape = __builtin_amdgcn_readfirstlane(tile.shape);
  const bool out_f16 = (s.kind & kSideOutF16) != 0;
  if (shape == kShape512x128)
    gemm_tile_body<512, 128, 4, 1, 2, false, IN, Any16>(p, tile, smem, s.beta_acc, s.beta_e, s.alpha_idx, s.diag_add, wave_id, out_f16);
  else if (shape == kShape256Diag)
    diag_tile_body<IN>(p, tile, smem, s.beta_acc, s.beta_e, s.alpha_idx, s.diag_add, wave_id);
  else
    gemm_tile_body<256, 256, 2, 2, 2, false, IN, Any16>(p, tile, smem, s.beta_acc, s.beta_e, s.alpha_idx, s.diag_add, wave_id, out_f16);
}
struct SharedArgs {
  GemmSide side[2];
  const GemmTile* tiles;
  int n_tiles;
};
__global__ __launch_bounds__(256, 1) void ns_pair_sym_kernel(SharedArgs args) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int wave_id = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  (void)args;
  for (int t = blockIdx.x;; t += gridDim.x) {
    // the arguments are read anew for every tile: kept in registers through a tile more would be spilled (29 vector registers are, around
    // the epilogues and in the tile loop, none of them in a K loop)
    const __attribute__((address_space(4))) SharedArgs* a = (const __attribute__((address_space(4))) SharedArgs*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(a));
    if (t >= a->n_tiles) break;
    const GemmTile tile = load_tile(a->tiles, t);
    const __attribute__((address_space(4))) GemmSide& side = a->side[__builtin_amdgcn_readfirstlane(tile.flags & kTileSecond) ? 1 : 0];
    GemmSide s;
    s.probs = side.probs; s.tiles = nullptr; s.n_tiles = 0;
    s.beta_acc = side.beta_acc; s.beta_e = side.beta_e; s.diag_add = side.diag_add;
    s.alpha_idx = side.alpha_idx; s.kind = side.kind; s.gain = 0.f;
    if (s.kind & kSideInF16) coarse_sym_tile<F16>(s, tile, smem, wave_id);
    else coarse_sym_tile<Bf16>(s, tile, smem, wave_id);
    __syncthreads();        // every wave has read its part of the LDS images: the next tile may overwrite them
  }
}

// Apply products of both sides in coarse tiles from one table, with bf16 operands: those of the first iteration, and of all iterations where
// nothing takes the Gram route.
__global__ __launch_bounds__(256, 1) void ns_pair_apply_kernel(SharedArgs args) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int wave_id = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  (void)args;
  for (int t = blockIdx.x;; t += gridDim.x) {
    const __attribute__((address_space(4))) SharedArgs* a = (const __attribute__((address_space(4))) SharedArgs*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(a));                  // see ns_pair_sym_kernel
    if (t >= a->n_tiles) break;
    const GemmTile tile = load_tile(a->tiles, t);
    const auto& s = a->side[(__builtin_amdgcn_readfirstlane(tile.flags) & kTileSecond) ? 1 : 0];
    const GemmProblem p = s.probs[tile.prob];
    const bool out_f16 = (s.kind & kSideOutF16) != 0;
    if (__builtin_amdgcn_readfirstlane(tile.shape) == kShape512x128)
      gemm_tile_body<512, 128, 4, 1, 2, true, Bf16, Any16>(p, tile, smem, s.beta_acc, s.beta_e, s.alpha_idx, s.diag_add, wave_id, out_f16);
    else
      gemm_tile_body<256, 256, 2, 2, 2, true, Bf16, Any16>(p, tile, smem, s.beta_acc, s.beta_e, s.alpha_idx, s.diag_add, wave_id, out_f16);
    __syncthreads();        // every wave has read its part of the LDS images: the next tile may overwrite them
  }
}

// An apply product in coarse tiles and, in the same launch, a product of the other side in 128-wide ones: the K-major tiles of 256
// leave compute units idle in their last round, and the side beside them would wait for a launch of its own.  The long tiles start first.
template <typename IN>
__global__ __launch_bounds__(256, 1) void ns_pair_beside_kernel(GemmSide x, GemmSide y, int blocks_x) {
  extern __shared__ __align__(16) unsigned char smem[];
  if ((int)blockIdx.x >= blocks_x) {
    const int t = (int)blockIdx.x - blocks_x;
    if (t >= y.n_tiles) return;
    const GemmTile tile = load_tile(y.tiles, t);
    const GemmProblem p = y.probs[tile.prob];
    with_operands(y.kind, [&](auto lkm, auto in, auto out) {
      gemm_ring128_body<decltype(lkm)::value, decltype(in), decltype(out)>(p, tile.r0 * kTileUnit, tile.c0 * kTileUnit, (tile.flags & kTileDiagonal) != 0, smem,
                                                                           y.beta_acc, y.beta_e, y.alpha_idx, 0.0, y.diag_add, (y.kind & kSideOutF16) != 0);
    });
    return;
  }
  const int t = (int)blockIdx.x;
  if (t >= x.n_tiles) return;
  const int wave_id = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const GemmTile tile = load_tile(x.tiles, t);
  const GemmProblem p = x.probs[tile.prob];
  const bool out_f16 = (x.kind & kSideOutF16) != 0;
  if (__builtin_amdgcn_readfirstlane(tile.shape) == kShape512x128)
    gemm_tile_body<512, 128, 4, 1, 2, true, IN, Any16>(p, tile, smem, x.beta_acc, x.beta_e, x.alpha_idx, x.diag_add, wave_id, out_f16);
  else
    gemm_tile_body<256, 256, 2, 2, 2, true, IN, Any16>(p, tile, smem, x.beta_acc, x.beta_e, x.alpha_idx, x.diag_add, wave_id, out_f16);
}

template <bool LKM, typename IN>
hipError_t setup_coarse() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&ns_pair_coarse_kernel<LKM, IN>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLds512);
}
template <bool LKM, typename IN>
void launch_coarse(int flags, const GemmSide& x, hipStream_t s) {
  const int grid = gemm_coarse_blocks();
  ns_pair_coarse_kernel<LKM, IN><<<(flags & kGemmPersistent) && x.n_tiles > grid ? grid : x.n_tiles, 256, (flags & kGemmStrips) ? kLds512 : kLds256, s>>>(
      x.probs, x.tiles, x.n_tiles, x.beta_acc, x.beta_e, x.alpha_idx, x.diag_add, (x.kind & kSideOutF16) != 0);
}

// a symmetric product writes what it reads
bool kinds_match(const GemmSide& p) { return (p.kind & kSideKMajor) || ((p.kind & kSideInF16) != 0) == ((p.kind & kSideOutF16) != 0); }

}  // namespace

hipError_t gemm_pair_setup() {
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&ns_pair_fine_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLds128);
  if (e == hipSuccess)
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&ns_pair_ring128_kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)(kLdsRing128 + kLdsFold64));
  if (e == hipSuccess)
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&ns_pair_tile64_kernel<kRing64, 3>), hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)(lds_ring64(kRing64) + kLdsFold64));
  if (e == hipSuccess)
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&ns_pair_tile64_kernel<kRing64Few, 2>), hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)(lds_ring64(kRing64Few) + kLdsFold64));
  if (e == hipSuccess)
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&ns_pair_sym_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLds512);
  if (e == hipSuccess)
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&ns_pair_apply_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLds512);
  if (e == hipSuccess)
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&ns_pair_beside_kernel<Bf16>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLds512);
  if (e == hipSuccess)
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&ns_pair_beside_kernel<F16>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLds512);
  if (e == hipSuccess) e = setup_coarse<true, Bf16>();
  if (e == hipSuccess) e = setup_coarse<false, F16>();
  if (e == hipSuccess) e = setup_coarse<true, F16>();
  return e;
}

hipError_t launch_gemm_beside(int flags, const GemmSide& x, const GemmSide& y, hipStream_t s) {
  if (x.n_tiles <= 0 || y.n_tiles <= 0 || !(x.kind & kSideKMajor) || !kinds_match(y) || x.alpha_idx == kAlphaFromPartials || y.alpha_idx == kAlphaFromPartials)
    return hipErrorInvalidValue;
  static_assert(kLdsRing128 <= kLds256, "every block of the launch gets the coarse tile's LDS");
  const int bx = (x.n_tiles + 7) / 8 * 8;
  const size_t lds = (flags & kGemmStrips) ? kLds512 : kLds256;
  if (x.kind & kSideInF16) ns_pair_beside_kernel<F16><<<bx + y.n_tiles, 256, lds, s>>>(x, y, bx);
  else ns_pair_beside_kernel<Bf16><<<bx + y.n_tiles, 256, lds, s>>>(x, y, bx);
  return hipGetLastError();
}

hipError_t launch_gemm_pair(int coarse, int flags, const GemmSide& x, const GemmSide& y, double eps, hipStream_t s) {
  if (x.n_tiles < 0 || y.n_tiles < 0) return hipErrorInvalidValue;
  if (x.n_tiles + y.n_tiles == 0) return hipSuccess;
  if (!kinds_match(x) || !kinds_match(y)) return hipErrorInvalidValue;
  const bool fold = x.alpha_idx == kAlphaFromPartials || y.alpha_idx == kAlphaFromPartials;
  if (fold && (coarse || !(flags & (kGemmQuarters | kGemmRing128)) || ((x.kind | y.kind) & kSideKMajor))) return hipErrorInvalidValue;
  const size_t fold_lds = fold ? kLdsFold64 : 0;
  if (coarse) {
    for (const GemmSide* p : {&x, &y}) {
      if (p->n_tiles == 0) continue;
      const bool f16 = (p->kind & kSideInF16) != 0;
      if (!(p->kind & (kSideInF16 | kSideOutF16))) {
        const hipError_t e = launch_gemm_bf16(1, flags, p->probs, p->tiles, p->n_tiles, p->beta_acc, p->beta_e, p->alpha_idx, eps, p->diag_add,
                                              (p->kind & kSideKMajor) != 0, 1, s);
        if (e != hipSuccess) return e;
        continue;
      }
      if (!(p->kind & kSideKMajor)) launch_coarse<false, F16>(flags, *p, s);
      else if (f16) launch_coarse<true, F16>(flags, *p, s);
      else launch_coarse<true, Bf16>(flags, *p, s);
    }
  } else if (flags & kGemmSixteenths) {
    const int bx = (x.n_tiles + 7) / 8 * 128;
    ns_pair_tile32_kernel<<<bx + (y.n_tiles + 7) / 8 * 128, 64, kLdsRing32, s>>>(x, y, bx, eps);
  } else if (flags & kGemmFewQuarters) {
    const int bx = (x.n_tiles + 7) / 8 * 32;
    ns_pair_tile64_kernel<kRing64Few, 2><<<bx + (y.n_tiles + 7) / 8 * 32, 256, lds_ring64(kRing64Few) + fold_lds, s>>>(x, y, bx, eps);
  } else if (flags & kGemmQuarters) {
    const int bx = (x.n_tiles + 7) / 8 * 32;
    ns_pair_tile64_kernel<kRing64, 3><<<bx + (y.n_tiles + 7) / 8 * 32, 256, lds_ring64(kRing64) + fold_lds, s>>>(x, y, bx, eps);
  } else if (flags & kGemmRing128) {
    const int bx = (x.n_tiles + 7) / 8 * 8;
    ns_pair_ring128_kernel<<<bx + y.n_tiles, 256, kLdsRing128 + fold_lds, s>>>(x, y, bx, eps);
  } else {
    const int bx = (x.n_tiles + 7) / 8 * 8;
    ns_pair_fine_kernel<<<bx + y.n_tiles, 256, kLds128, s>>>(x, y, bx);
  }
  return hipGetLastError();
}

hipError_t launch_gemm_shared(int flags, const GemmSide& x, const GemmSide& y, const GemmTile* tiles, int n_tiles, hipStream_t s) {
  if (n_tiles <= 0) return hipSuccess;
  const bool apply = (x.kind & kSideKMajor) != 0;
  if (apply != ((y.kind & kSideKMajor) != 0) || (apply && ((x.kind | y.kind) & kSideInF16)) || x.alpha_idx == kAlphaFromPartials || y.alpha_idx == kAlphaFromPartials)
    return hipErrorInvalidValue;
  const int grid = (flags & kGemmPersistent) && n_tiles > gemm_coarse_blocks() ? gemm_coarse_blocks() : n_tiles;
  const size_t lds = (flags & kGemmStrips) ? kLds512 : kLds256;
  const SharedArgs args{{x, y}, tiles, n_tiles};
  if (apply) ns_pair_apply_kernel<<<grid, 256, lds, s>>>(args);
  else ns_pair_sym_kernel<<<grid, 256, lds, s>>>(args);
  return hipGetLastError();
}

}  // namespace muon
