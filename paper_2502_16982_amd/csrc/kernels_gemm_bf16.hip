// bf16 Newton-Schulz products for gfx950 (Eq. 2 of the paper): grouped GEMMs
//     T[i][j] = sum_k L[i][k] * R[j][k]          (bf16 operands, fp32 accumulation on the matrix cores)
// with a fused epilogue  val = alpha * (beta_acc * acc + beta_e * E[i][j]) (+ a constant on the diagonal), storing
// T^T (cheap: it is the accumulator layout) and/or T.  R is always contiguous along k; L either contiguous along k
// or K-major (element (i, k) at L[k * ldl + i]).  With ONE row-major copy of the iterate X (m x n):
//     Gram       A  = X X^T                L = R = X                   (symmetric output)
//     polynomial B' = b A + c A A + a I    L = R = A                   (A symmetric; the a X term of the apply
//                                                                       product travels in B's diagonal)
//     apply      T  = X'^T = X^T B'        L = X read K-major, R = B'  (stores T^T = X' row-major; T itself only
//                                                                       where O is wanted transposed)
// Operands are zero-padded to whole tiles by the producer, so the kernel has no edge handling.
// Split operands: every matrix is the sum of PL = 2 or 3 bf16 arrays ("planes", plane q at element offset q * plane stride
// from the base pointer), each holding what the planes before it left of the fp32 value after rounding to bf16, i.e. about
// 2^-8 of its predecessor.  A product of two such sums is taken over the plane pairs (i, j) with i + j < PL - the pairs left
// out are below 2^(-8 PL) of the result - and its fp32 result is split into planes again (gemm_planes.h).
//
// Design for CDNA4:
//  * v_mfma_f32_32x32x16_bf16 (the 16x16x32 form runs at half the rate on this chip), wave tile = FM x FN
//    MFMA tiles, accumulators stay in registers for the whole K loop.
//  * K is consumed in 64-wide slabs, i.e. one 128-byte line per row: measured on this chip, the L1 hands a
//    compute unit ~57 B/clk when 8 lanes ask for a whole line and only ~26 B/clk for half lines.
//    Global memory -> LDS goes through the LDS-DMA path (global_load_lds_dwordx4): no staging registers, no
//    ds_write instructions.  A wave-level DMA instruction fills 1 KB of LDS contiguously (lane i -> byte 16*i),
//    i.e. 8 rows of 128 B; the 16-byte chunks of a row are XOR-swizzled by (row/2)%8 - each lane simply fetches
//    the global chunk that belongs in its slot - so that the 16 lanes served together by a ds_read_b128
//    fragment read hit 16 distinct bank groups (the bank-conflict counter reads zero).
//  * The LDS stages form a ring; a slab is requested one whole iteration (64 MFMAs per wave for the 256x256
//    tile) before it is needed.  One s_waitcnt + s_barrier per slab, placed in front of the last k-step so
//    that the next slab's first fragments are already being read while that k-step's MFMAs execute.
//  * Epilogue: the (transposed) addend tile is DMA-ed into LDS with coalesced 16-byte requests, each lane
//    combines it with its accumulators (fp32 math, one v_cvt_pk_bf16_f32 rounding), and results leave through
//    swizzled LDS images so that both the tile and its transpose are written with full 16-byte-per-lane
//    coalesced stores; the second orientation comes from a 2-MFMA transpose per 32x32 tile.
#include "gemm_tile256.h"
#include "gemm_planes.h"
#include "gemm_tile64.h"
#include "gemm_ring128.h"

namespace muon {
namespace {

// ---- kernels.  Fine launch: 128 x 128 tiles, two blocks per compute unit.  Coarse launch: one block per compute
// unit, each block running the shape its table entry names - 256 x 256 (2 x 2 waves) or 512 x 128 (4 x 1 waves; the
// 128-wide strips that an odd multiple of 128 leaves beside the 256-tiles).  Both coarse shapes give every wave a
// 128 x 128 tile, so they share register budget, MFMA schedule and per-wave LDS traffic, and a launch mixes them freely:
// the strips fill compute units next to the 256-tiles of the same product instead of running as a launch of their own.
constexpr size_t kLds128 = TileCfg<128, 128>::lds_bytes(2);
constexpr size_t lds_quarters(int planes) { return planes > 1 ? planes_lds(64, planes_ring(64, planes)) : lds_ring64(kRing64); }
constexpr size_t lds_few_quarters(int planes) { return planes > 1 ? planes_lds(64, kPlanesRingFew) : lds_ring64(kRing64Few); }
constexpr size_t lds_fine(int planes) { return planes > 1 ? planes_lds(128, planes_ring(128, planes)) : kLds128; }
constexpr size_t lds_coarse(bool kmajor, int planes) { return planes_lds(128, planes_ring_coarse(kmajor, planes)); }
constexpr size_t kLds256 = TileCfg<256, 256>::lds_bytes(2);
constexpr size_t kLds512 = TileCfg<512, 128>::lds_bytes(2);
constexpr int kMaxPlanes = 3;

template <bool LKM, int PL>
__global__ __launch_bounds__(256, PL == 3 ? 1 : 2) void ns_gemm_bf16_fine_kernel(const GemmProblem* __restrict__ probs,
                                                                    const GemmTile* __restrict__ tiles, float beta_acc,
                                                                    float beta_e, int alpha_idx, float diag_add) {
  extern __shared__ __align__(16) unsigned char smem[];
  const GemmTile tile = load_tile(tiles, blockIdx.x);
  const GemmProblem p = probs[tile.prob];
  if constexpr (PL > 1)
    planes_tile<128, planes_ring(128, PL), LKM, PL>(p, tile.r0 * kTileUnit, tile.c0 * kTileUnit, (tile.flags & kTileDiagonal) != 0, smem, beta_acc, beta_e,
                              alpha_idx, 0.0);
  else
    gemm_tile_body<128, 128, 2, 2, 2, LKM>(p, tile, smem, beta_acc, beta_e, alpha_idx, diag_add,
                                               __builtin_amdgcn_readfirstlane(threadIdx.x >> 6));
}

// Each table entry as one block with a compute unit to itself.
template <bool LKM>
__global__ __launch_bounds__(256, 1) void ns_ring128_bf16_kernel(const GemmProblem* __restrict__ probs, const GemmTile* __restrict__ tiles,
                                                                 float beta_acc, float beta_e, int alpha_idx, double eps, float diag_add) {
  extern __shared__ __align__(16) unsigned char smem[];
  const GemmTile tile = load_tile(tiles, blockIdx.x);
  const GemmProblem p = probs[tile.prob];
  gemm_ring128_body<LKM>(p, tile.r0 * kTileUnit, tile.c0 * kTileUnit, (tile.flags & kTileDiagonal) != 0, smem, beta_acc, beta_e, alpha_idx, eps,
                         diag_add);
}

// Each 128 x 128 table entry as four blocks of 64 x 64.  Block b: entry 8 (b / 32) + b % 8, so that an entry's quarters
// run on the die its entry is dealt to; quarter (b / 8) % 4.
template <bool LKM, int PL>
__global__ __launch_bounds__(256, PL == 3 ? 2 : 3) void ns_tile64_gemm_bf16_kernel(const GemmProblem* __restrict__ probs,
                                                                   const GemmTile* __restrict__ tiles, int n_tiles, float beta_acc,
                                                                   float beta_e, int alpha_idx, double eps, float diag_add) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int t = (int)(blockIdx.x >> 5) * 8 + (int)(blockIdx.x & 7), quarter = (int)(blockIdx.x >> 3) & 3;
  if (t >= n_tiles) return;
  const GemmTile tile = load_tile(tiles, t);
  const bool on_diag = (tile.flags & kTileDiagonal) != 0;
  if (on_diag && quarter == 2) return;           // below the diagonal: the mirror image of quarter 1
  const GemmProblem p = probs[tile.prob];
  const int row0 = tile.r0 * kTileUnit + 64 * (quarter >> 1), col0 = tile.c0 * kTileUnit + 64 * (quarter & 1);
  if constexpr (PL > 1) planes_tile<64, planes_ring(64, PL), LKM, PL>(p, row0, col0, on_diag && quarter != 1, smem, beta_acc, beta_e, alpha_idx, eps);
  else gemm_tile64_body<LKM, 4, kRing64>(p, row0, col0, on_diag && quarter != 1, smem, beta_acc, beta_e, alpha_idx, eps, diag_add);
}

// The same with a ring of four stages: two blocks fit a compute unit instead of three.
template <bool LKM, int PL>
__global__ __launch_bounds__(256, 2) void ns_ring4_gemm_bf16_kernel(const GemmProblem* __restrict__ probs, const GemmTile* __restrict__ tiles,
                                                                    int n_tiles, float beta_acc, float beta_e, int alpha_idx, double eps,
                                                                    float diag_add) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int t = (int)(blockIdx.x >> 5) * 8 + (int)(blockIdx.x & 7), quarter = (int)(blockIdx.x >> 3) & 3;
  if (t >= n_tiles) return;
  const GemmTile tile = load_tile(tiles, t);
  const bool on_diag = (tile.flags & kTileDiagonal) != 0;
  if (on_diag && quarter == 2) return;
  const GemmProblem p = probs[tile.prob];
  const int row0 = tile.r0 * kTileUnit + 64 * (quarter >> 1), col0 = tile.c0 * kTileUnit + 64 * (quarter & 1);
  if constexpr (PL > 1) planes_tile<64, kPlanesRingFew, LKM, PL>(p, row0, col0, on_diag && quarter != 1, smem, beta_acc, beta_e, alpha_idx, eps);
  else gemm_tile64_body<LKM, 4, kRing64Few>(p, row0, col0, on_diag && quarter != 1, smem, beta_acc, beta_e, alpha_idx, eps, diag_add);
}

// Each entry as sixteen blocks of one wave and 32 x 32.  Block b: entry 8 (b / 128) + b % 8, sixteenth (b / 8) % 16.
template <bool LKM>
__global__ __launch_bounds__(64) void ns_tile32_gemm_bf16_kernel(const GemmProblem* __restrict__ probs, const GemmTile* __restrict__ tiles,
                                                                 int n_tiles, float beta_acc, float beta_e, int alpha_idx, double eps,
                                                                 float diag_add) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int t = (int)(blockIdx.x >> 7) * 8 + (int)(blockIdx.x & 7), part = (int)(blockIdx.x >> 3) & 15;
  if (t >= n_tiles) return;
  const GemmTile tile = load_tile(tiles, t);
  const bool on_diag = (tile.flags & kTileDiagonal) != 0;
  if (on_diag && (part >> 2) > (part & 3)) return;   // below the diagonal: a mirror image
  const GemmProblem p = probs[tile.prob];
  gemm_tile64_body<LKM, 1, kRing32>(p, tile.r0 * kTileUnit + 32 * (part >> 2), tile.c0 * kTileUnit + 32 * (part & 3),
                           on_diag && (part >> 2) == (part & 3), smem, beta_acc, beta_e, alpha_idx, eps, diag_add);
}

// Block b works through table entries b, b + gridDim.x, ...  Launched with one block per tile, or persistent: one
// block per compute unit (a multiple of the 8 dies, so an entry still runs on die index % 8); a persistent block that
// goes on to its next tile neither waits for its stores to drain nor is re-dispatched, and its next tile's first
// operand requests overlap both (measured +2 % on the MoE bank; with tiles of mixed K the static dealing loses that
// again, so such launches stay one block per tile).
// With several planes every entry is four blocks of 128 x 128 on the entry's die, none of them persistent: a 256-wide tile has
// no registers for the planes' fragments (gemm_planes.h holds both sides' times).
template <bool LKM, int PL>
__global__ __launch_bounds__(256, PL == 2 && LKM ? 2 : 1) void ns_gemm_bf16_kernel(const GemmProblem* __restrict__ probs,
                                                               const GemmTile* __restrict__ tiles, int n_tiles, float beta_acc,
                                                               float beta_e, int alpha_idx, float diag_add) {
  extern __shared__ __align__(16) unsigned char smem[];
  if constexpr (PL > 1) {
    const int t = (int)(blockIdx.x >> 5) * 8 + (int)(blockIdx.x & 7), quarter = (int)(blockIdx.x >> 3) & 3;
    if (t >= n_tiles) return;
    const GemmTile tile = load_tile(tiles, t);
    const bool strip = tile.shape == kShape512x128;
    const GemmProblem p = probs[tile.prob];
    const int row0 = tile.r0 * kTileUnit + 128 * (strip ? quarter : quarter >> 1), col0 = tile.c0 * kTileUnit + 128 * (strip ? 0 : quarter & 1);
    if (p.symmetric && row0 > col0) return;      // below the diagonal: a mirror image
    // the last strip of a column is shifted up to end at the edge: what its neighbour computes too is left to that
    const int own_row = strip ? (tile.r0 * kTileUnit + kShapeRows[kShape512x128] - 1) / kShapeRows[kShape512x128] * kShapeRows[kShape512x128] : 0;
    if (row0 < own_row) return;
    planes_tile<128, planes_ring_coarse(LKM, PL), LKM, PL>(p, row0, col0, p.symmetric && row0 == col0, smem, beta_acc, beta_e, alpha_idx, 0.0);
  } else {
    const int wave_id = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (int t = blockIdx.x; t < n_tiles; t += gridDim.x) {
      const GemmTile tile = load_tile(tiles, t);
      const GemmProblem p = probs[tile.prob];
      const int shape = __builtin_amdgcn_readfirstlane(tile.shape);
      if (shape == kShape512x128) {
        gemm_tile_body<512, 128, 4, 1, 2, LKM>(p, tile, smem, beta_acc, beta_e, alpha_idx, diag_add, wave_id);
      } else if (!LKM && shape == kShape256Diag) {
        if constexpr (!LKM) diag_tile_body(p, tile, smem, beta_acc, beta_e, alpha_idx, diag_add, wave_id);
      } else {
        gemm_tile_body<256, 256, 2, 2, 2, LKM>(p, tile, smem, beta_acc, beta_e, alpha_idx, diag_add, wave_id);
      }
      __syncthreads();        // every wave has read its part of the LDS images: the next tile may overwrite them
    }
  }
}

int g_coarse_grid = 0;      // blocks of a coarse launch: one per compute unit (set by gemm_setup)

template <bool LKM, int PL>
hipError_t setup_pair() {
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&ns_gemm_bf16_fine_kernel<LKM, PL>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_fine(PL));
  if (e == hipSuccess)
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&ns_tile64_gemm_bf16_kernel<LKM, PL>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)(lds_quarters(PL) + kLdsFold64));
  if (e == hipSuccess)
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&ns_ring4_gemm_bf16_kernel<LKM, PL>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)(lds_few_quarters(PL) + kLdsFold64));
  if (e == hipSuccess && PL == 1)
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&ns_ring128_bf16_kernel<LKM>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)(kLdsRing128 + kLdsFold64));
  if (e != hipSuccess) return e;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&ns_gemm_bf16_kernel<LKM, PL>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)(PL > 1 ? lds_coarse(LKM, PL) : kLds512));
}

template <bool LKM, int PL>
void launch_one(int coarse, int flags, const GemmProblem* probs, const GemmTile* tiles, int n_tiles, float beta_acc,
                float beta_e, int alpha_idx, double eps, float diag_add, hipStream_t s) {
  if (PL == 1 && !coarse && (flags & kGemmSixteenths))
    ns_tile32_gemm_bf16_kernel<LKM><<<(n_tiles + 7) / 8 * 128, 64, kLdsRing32, s>>>(probs, tiles, n_tiles, beta_acc, beta_e, alpha_idx,
                                                                                    eps, diag_add);
  else if (!coarse && (flags & kGemmFewQuarters))
    ns_ring4_gemm_bf16_kernel<LKM, PL><<<(n_tiles + 7) / 8 * 32, 256,
                                         lds_few_quarters(PL) + (alpha_idx == kAlphaFromPartials ? kLdsFold64 : 0), s>>>(
        probs, tiles, n_tiles, beta_acc, beta_e, alpha_idx, eps, diag_add);
  else if (!coarse && (flags & kGemmQuarters))
    ns_tile64_gemm_bf16_kernel<LKM, PL><<<(n_tiles + 7) / 8 * 32, 256,
                                          lds_quarters(PL) + (alpha_idx == kAlphaFromPartials ? kLdsFold64 : 0), s>>>(
        probs, tiles, n_tiles, beta_acc, beta_e, alpha_idx, eps, diag_add);
  else if (PL == 1 && !coarse && (flags & kGemmRing128))
    ns_ring128_bf16_kernel<LKM><<<n_tiles, 256, kLdsRing128 + (alpha_idx == kAlphaFromPartials ? kLdsFold64 : 0), s>>>(probs, tiles, beta_acc, beta_e,
                                                                                                                     alpha_idx, eps, diag_add);
  else if (!coarse)
    ns_gemm_bf16_fine_kernel<LKM, PL><<<n_tiles, 256, lds_fine(PL), s>>>(probs, tiles, beta_acc, beta_e, alpha_idx, diag_add);
  else
    ns_gemm_bf16_kernel<LKM, PL><<<PL > 1 ? (n_tiles + 7) / 8 * 32 : (flags & kGemmPersistent) && n_tiles > g_coarse_grid ? g_coarse_grid : n_tiles,
                                   256, PL > 1 ? lds_coarse(LKM, PL) : (flags & kGemmStrips) ? kLds512 : kLds256, s>>>(
        probs, tiles, n_tiles, beta_acc, beta_e, alpha_idx, diag_add);
}

}  // namespace

int gemm_coarse_blocks() { return g_coarse_grid; }

hipError_t gemm_setup() {
  int dev = 0, cus = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  g_coarse_grid = cus > 0 ? cus : 256;
  // the kernels' attributes stay set: once per device is enough (two threads that get here together set them twice)
  static std::atomic<uint64_t> done{0};
  const uint64_t bit = dev < 64 ? uint64_t{1} << dev : 0;
  if (done.load(std::memory_order_acquire) & bit) return hipSuccess;
  e = setup_pair<false, 1>();
  if (e == hipSuccess) e = setup_pair<true, 1>();
  if (e == hipSuccess) e = setup_pair<false, 2>();
  if (e == hipSuccess) e = setup_pair<true, 2>();
  if (e == hipSuccess) e = setup_pair<false, 3>();
  if (e == hipSuccess) e = setup_pair<true, 3>();
  if (e == hipSuccess) e = gemm_pair_setup();
  if (e == hipSuccess) e = gemm_f32_setup();
  if (e == hipSuccess) done.fetch_or(bit, std::memory_order_release);
  return e;
}

hipError_t launch_gemm_bf16(int coarse, int flags, const GemmProblem* probs, const GemmTile* tiles, int n_tiles, float beta_acc,
                            float beta_e, int alpha_idx, double eps, float diag_add, int l_kmajor, int planes, hipStream_t s) {
  if (n_tiles <= 0) return hipSuccess;
  if (planes < 1 || planes > kMaxPlanes) return hipErrorInvalidValue;
  if (alpha_idx == kAlphaFromPartials && (coarse || l_kmajor || !(flags & (kGemmQuarters | kGemmRing128)))) return hipErrorInvalidValue;
#define MUON_GEMM_CASE(K, P)                                                                                     \
  if ((l_kmajor != 0) == K && planes == P) launch_one<K, P>(coarse, flags, probs, tiles, n_tiles, beta_acc, beta_e, alpha_idx, eps, diag_add, s)
  MUON_GEMM_CASE(false, 1);
  MUON_GEMM_CASE(true, 1);
  MUON_GEMM_CASE(false, 2);
  MUON_GEMM_CASE(true, 2);
  MUON_GEMM_CASE(false, 3);
  MUON_GEMM_CASE(true, 3);
#undef MUON_GEMM_CASE
  return hipGetLastError();
}

}  // namespace muon
