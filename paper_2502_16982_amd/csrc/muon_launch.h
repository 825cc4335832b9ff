// Host-callable launchers of the HIP kernels (internal to the library).
#pragma once
#include <hip/hip_runtime.h>

#include "adamw_batch.h"
#include "muon_tables.h"

namespace muon {

// A table entry through whole-dword loads, so that they are scalar loads: the sub-dword fields would otherwise come
// through a vector load, and the wait for it is a wait for every store of the block's previous tile as well.
__device__ __forceinline__ GemmTile load_tile(const GemmTile* __restrict__ tiles, int t) {
  static_assert(sizeof(GemmTile) == 12, "three dwords");
  const uint32_t* w = reinterpret_cast<const uint32_t*>(tiles) + 3 * (size_t)t;
  const uint32_t w0 = w[0], w1 = w[1], w2 = w[2];
  GemmTile r;
  r.prob = (int32_t)w0;
  r.r0 = (uint16_t)(w1 & 0xffffu);
  r.c0 = (uint16_t)(w1 >> 16);
  r.shape = (uint8_t)(w2 & 0xffu);
  r.flags = (uint8_t)((w2 >> 8) & 0xffu);
  r.pad_ = 0;
  return r;
}

// Sum of n floats in double by the 256 threads of a block, in the order of the norm's own kernel, returned to every lane
// (red: 256 doubles of LDS).  Contains one barrier.
__device__ __forceinline__ double block_sum_f64(const float* __restrict__ v, int n, double* red) {
  double acc = 0.0;
  for (int i = threadIdx.x; i < n; i += 256) acc += (double)v[i];
  red[threadIdx.x] = acc;
  __syncthreads();
  const int l = threadIdx.x & 63;
  double t = (red[l] + red[l + 128]) + (red[l + 64] + red[l + 192]);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) t += __shfl_xor(t, off, 64);
  return t;
}
// The same sum in the same order by one wave.
__device__ __forceinline__ double wave_sum_f64(const float* __restrict__ v, int n) {
  const int l = threadIdx.x & 63;
  double acc[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    acc[q] = 0.0;
    for (int i = l + 64 * q; i < n; i += 256) acc[q] += (double)v[i];
  }
  double t = (acc[0] + acc[2]) + (acc[1] + acc[3]);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) t += __shfl_xor(t, off, 64);
  return t;
}
// a2: 1/(sqrt(sum) + eps) and its square from the sum of squares of U.  An all-zero U with eps = 0 would give inf; X is all
// zero then, and 0 * inf must not appear.
__device__ __forceinline__ void norm_scalars(double sum, double eps, float* s, float* s2) {
  const double inv = 1.0 / (sqrt(sum) + eps);
  const bool ok = sum > 0.0 || eps > 0.0;
  *s = ok ? (float)inv : 0.f;
  *s2 = ok ? (float)(inv * inv) : 0.f;
}
// They go to scal[0] and scal[1].  gain > 0 (Gram route: no iteration sequence of the launch makes X larger than that many times): where
// eps leaves X so small that it stays below 4, X between the first and the last iteration is kept 2^k times as large, up to 4, well inside
// f16; scal[0] then carries 2^k, [2] and [3] are 2^-2k and 2^-k.
__device__ __forceinline__ void store_norm(float* scal, double sum, double eps, float gain, float s, float s2) {
  if (gain > 0.f) {
    const double x = sqrt(sum), most = x / (x + eps) * (double)gain;           // (all zero: any scale will do)
    const int k = most < 4.0 && most > 0.0 ? min(1 - ilogb(most), 40) : 0;
    s *= ldexpf(1.f, k);
    scal[2] = ldexpf(1.f, -2 * k);
    scal[3] = ldexpf(1.f, -k);
  }
  scal[0] = s;
  scal[1] = s2;
}

// One-time per-process kernel attribute setup (large dynamic LDS).  Returns a hipError_t.
hipError_t gemm_setup();
// Blocks of a persistent coarse GEMM launch = compute units of the device gemm_setup ran on (0 before it).
int gemm_coarse_blocks();

// a1-a3: momentum, sum of squares, cast + orient.  both_layouts != 0: U goes to X and Xt[0] (one holds U, the other
// U^T); 0: only X (the orientation with rows <= cols) is written.  One block per EwTile.
// pack != null: the pointers come as a kernel argument and the pass leaves them in `ptrs` for the kernels behind it.
constexpr int kPackSlots = 64;
struct PtrPack {
  MatPtrs p[kPackSlots];
};
hipError_t launch_momentum_norm_cast(const MatDesc* mats, MatPtrs* ptrs, const PtrPack* pack, const EwTile* tiles, int n_tiles,
                                     float mu, int nesterov, int both_layouts, int ns_dtype, hipStream_t s);

// a2 second stage: fixed-order sum of the partials of each matrix, s = 1/(sqrt(sum)+eps).
// gram_gain: store_norm's gain for matrices of the Gram route (0: they are iterated as Eq. 2 is written).
hipError_t launch_norm_finalize(const MatDesc* mats, int first_mat, int n_mats, double eps, float gram_gain, hipStream_t s);

// a4-a6: grouped NT GEMM with fused epilogue.  alpha_idx: -1 none, 0 .. 3 -> that scal[], kAlphaFromPartials (first
// Gram product, kGemmQuarters and kGemmRing128 launches only) -> what scal[1] has to be, from the partial sums of squares and eps; the block
// of the first tile leaves them behind (store_norm).  diag_add: constant
// added to the diagonal of the outputs of problems that ask for it (GemmProblem::diag_add), bf16 kernel only.
// coarse: 0 = every tile of the table is 128 x 128 (two blocks per compute unit); 1 = the table mixes 256 x 256 and,
// with kGemmStrips in `flags`, 512 x 128 tiles (one block per compute unit; the flag selects the larger LDS
// allocation).  kGemmPersistent: one block per compute unit works through the table with stride gridDim (for launches
// whose tiles run K loops of nearly the same length, which the planner balances statically; with a wide spread of K
// the hardware's dynamic block dispatch does better).
// kGemmQuarters (coarse = 0): every entry of the table runs as four blocks, one per quarter of it.  kGemmFewQuarters
// (with kGemmQuarters): with a longer ring; kGemmSixteenths (plain bf16, with kGemmQuarters): as sixteen blocks of one wave.
// kGemmRing128 (coarse = 0, plain bf16, K >= 256): one block per entry, with a compute unit to itself.
// kGemmLongK (fp32): needed where a problem of the launch has K > kF32LongK.
// l_kmajor: every problem of the launch stores its L operand K-major (element (i, k) at L[k * ldl + i]).
// planes: 1 = plain bf16; 2 or 3 = every matrix is a sum of that many bf16 planes (GemmProblem::*_plane strides); entries of a
// coarse table then run as four 128 x 128 blocks each.
constexpr int kAlphaFromPartials = 4;
constexpr int kGemmStrips = 1, kGemmPersistent = 2, kGemmQuarters = 4, kGemmLongK = 8, kGemmSixteenths = 16, kGemmFewQuarters = 32, kGemmRing128 = 64;
hipError_t launch_gemm_bf16(int coarse, int flags, const GemmProblem* probs, const GemmTile* tiles, int n_tiles,
                            float beta_acc, float beta_e, int alpha_idx, double eps, float diag_add, int l_kmajor, int planes,
                            hipStream_t s);
// Two products in one launch (kernels_gemm_pair.hip), either of them empty (n_tiles = 0).  coarse, flags, eps: as above; in a
// coarse launch both sides' tables are coarse ones.
struct GemmSide {
  const GemmProblem* probs;
  const GemmTile* tiles;
  int n_tiles;
  float beta_acc, beta_e, diag_add;
  int alpha_idx;
  int kind;           // kSide*: operand layout, type of the operands and the addend, type of the results
  float gain;         // kAlphaFromPartials: store_norm's
};
constexpr int kSideKMajor = 1, kSideInF16 = 2, kSideOutF16 = 4;
hipError_t gemm_pair_setup();
hipError_t launch_gemm_pair(int coarse, int flags, const GemmSide& x, const GemmSide& y, double eps, hipStream_t s);
// x, an apply product in coarse tiles, and y in 128-wide ones (K >= 256), one block per compute unit.
hipError_t launch_gemm_beside(int flags, const GemmSide& x, const GemmSide& y, hipStream_t s);
// Coarse symmetric products of both, or apply products with bf16 operands, from one table; the sides' own tables are not used.
hipError_t launch_gemm_shared(int flags, const GemmSide& x, const GemmSide& y, const GemmTile* tiles, int n_tiles, hipStream_t s);
hipError_t gemm_f32_setup();
// tail: the last entries of a table of whole ones, as many, that run in quarters in a launch of their own.
hipError_t launch_gemm_f32(int flags, int tail, const GemmProblem* probs, const GemmTile* tiles, int n_tiles,
                           float beta_acc, float beta_e, int alpha_idx, double eps, hipStream_t s);

// a8: W <- W - lr*(scale*O + wd*W); also leaves per-tile sums of O^2 in the partials.
// o_sel: where O sits in W's orientation: bit 0 picks Xt[0] / Xt[1] for matrices iterated on their transpose, bit 1
// picks X (0) or Xt[0] (1) for the others; use_s: multiply O by scal[0] (only when no Newton-Schulz iteration ran).
// scale_mode: 0 factor = rms_scale*sqrt(max(A,B)); 1 factor = rms_scale*sqrt_hidden; 2 factor = rms_scale*scal[2]
// (scal[2] = 1/RMS of the stored O, left there by launch_update_rms(..., to_scal = 1)).
// stream_w: the streaming hint on accesses to bf16 weights (for rows that end on whole lines).
hipError_t launch_apply_update(const MatDesc* mats, const MatPtrs* ptrs, const EwTile* tiles, int n_tiles,
                               float lr, float wd, float rms_scale, int scale_mode, float sqrt_hidden, int o_sel,
                               int use_s, int stream_w, int ns_dtype, hipStream_t s);

// Per-tile sums of O^2 into the partials, without touching W (first pass of the "Update Norm" variant).
hipError_t launch_update_sumsq(const MatDesc* mats, const EwTile* tiles, int n_tiles, int o_sel, int ns_dtype, hipStream_t s);

// From the per-tile sums of O^2: to_scal = 0 writes sqrt(mean(O^2)) per matrix to out; to_scal = 1 writes
// 1/sqrt(mean(stored O^2)) (0 when O = 0) to scal[2].
hipError_t launch_update_rms(const MatDesc* mats, int first_mat, int n_mats, int use_s, int to_scal, float* out, hipStream_t s);

// Test hook: O of one matrix -> dst (rows x cols contiguous).
hipError_t launch_read_update(const MatDesc* mats, int mat, int o_sel, int use_s, int ns_dtype, void* dst,
                              int dst_dtype, hipStream_t s);

// AdamW (non-matrix parameters): one launch over the pieces of a batch (adamw_batch.h).
hipError_t launch_adamw(const AdamwBatch& batch, int n_blocks, float lr, float wd, float beta1, float beta2, float eps,
                        float inv_bc1, float inv_bc2, hipStream_t s);

}  // namespace muon
