// fp32 Newton-Schulz products for gfx950 (Eq. 2 of the paper), used when the caller asks for fp32 iteration
// arithmetic: grouped "NT" GEMM  C[i][j] = sum_k L[i][k] * R[j][k]  with the same problem/tile tables and
// fused epilogue  val = alpha * (beta_acc * acc + beta_e * Et[j][i])  as the bf16 MFMA kernel.
//
// The products run on v_mfma_f32_32x32x2_f32 (fp32 operands, fp32 accumulation; twice the rate of unpacked fp32 FMAs,
// and a fragment read from LDS feeds 32 multiply-adds instead of 4).  Operands come through the LDS-DMA path into a ring
// of slabs of 32 k (one 128-byte line per row, 16-byte chunks XOR-swizzled by (row / 2) % 8) that are waited for with a
// partial s_waitcnt vmcnt; half a slab's fragments are read while the other half is multiplied.  Two forms:
//  * whole:    a block owns a 64 x 64 table entry, four waves of 32 x 32, all of K, one barrier per slab.  A slab is 16 KB
//              for 1024 clocks of MFMAs per wave: bound by the matrix cores.
//  * quarters: an entry is four blocks of 32 x 32 whose four waves take every fourth slab each, from a ring of their own
//              (no barrier before the partial results are added up).  For launches with few entries: four times as many
//              blocks and a K loop a quarter as long, at twice the operand traffic.
// Measured, us per step of one matrix (four of them) when the two forms came in, a 64 x 64 tile of FMAs without prefetch /
// whole / quarters: 128 x 256 244 / 125 / 78, 512 x 512 555 / 241 / 124 (575 / 257 / 241), 1024 x 1024 1016 / 390 / 346
// (1694 / 982 / 989).  Now 128 x 256 59 (with the elementwise passes and the norm of today), 512 x 512 105 (207), 1024 x 1024 313
// (967: apply product 78 us = 110 TFLOP/s of the 157 the fp32 matrix instructions can do).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "muon_launch.h"

namespace muon {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(1))) void* gptr;
typedef __attribute__((address_space(3))) void* lptr;

constexpr int BKF = 32;                          // K slab in elements: one 128-byte line per row
constexpr int ROWF = 128;                        // bytes per LDS row
constexpr int kImgPitch = 36;                    // floats per row of the 32 x 32 result images (conflict-free 16-byte writes)

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// Two 8-wide k-steps of a wave's fragments, read by assembly (in front of an LDS read of its own the compiler puts a
// wait for all vector memory, the slabs in flight included); the wait takes the registers as read-write operands, so
// every MFMA on them depends on it.
struct HalfSlab {
  f32x4 a[2], b[2];
};
__device__ __forceinline__ void read_half(HalfSlab& f, unsigned a0, unsigned a1, unsigned b0, unsigned b1) {
  asm volatile("ds_read_b128 %0, %1" : "=v"(f.a[0]) : "v"(a0) : "memory");
  asm volatile("ds_read_b128 %0, %1" : "=v"(f.b[0]) : "v"(b0) : "memory");
  asm volatile("ds_read_b128 %0, %1" : "=v"(f.a[1]) : "v"(a1) : "memory");
  asm volatile("ds_read_b128 %0, %1" : "=v"(f.b[1]) : "v"(b1) : "memory");
}
__device__ __forceinline__ void land_half(HalfSlab& f) {
  asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(f.a[0]), "+v"(f.b[0]), "+v"(f.a[1]), "+v"(f.b[1]) : : "memory");
}

// two slabs per wave's own ring leave room for two blocks of quarters on a compute unit (three: 1024^2 -> 408 instead of 346 us)
constexpr int ring_of(bool quarters) { return quarters ? 2 : 3; }
constexpr size_t stage_bytes(bool quarters) { return quarters ? 4 * 64 * ROWF : 128 * ROWF; }
constexpr size_t kLdsFold = 256 * sizeof(double);            // scratch behind the rings for the folded norm
constexpr size_t lds_bytes(bool quarters) { return ring_of(quarters) * stage_bytes(quarters); }

// Barrier for what is in LDS: unlike __syncthreads it does not wait for loads from memory that are on their way.
__device__ __forceinline__ void meet() {
  asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" : : : "memory");
}

template <bool Q, bool LONG>
__global__ __launch_bounds__(256, Q || LONG ? 2 : 3) void ns_gemm_f32_kernel(const GemmProblem* __restrict__ probs,
                                                              const GemmTile* __restrict__ tiles, int n_tiles, float beta_acc,
                                                              float beta_e, int alpha_idx, double eps) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int NST = ring_of(Q), NLOAD = Q ? 8 : 4;            // stages, 1 KB requests per wave and slab
  constexpr int ROWS = Q ? 32 : 64;                             // rows of each operand in a stage
  static_assert(lds_bytes(Q) >= 4 * 32 * kImgPitch * sizeof(float) && NST == (Q ? 2 : 3), "ring shape");
  // quarters: block b works on entry 8 (b / 32) + b % 8 (so that an entry's blocks run on the die it is dealt to)
  const int t = Q ? (int)(blockIdx.x >> 5) * 8 + (int)(blockIdx.x & 7) : (int)blockIdx.x;
  const int quarter = Q ? (int)(blockIdx.x >> 3) & 3 : 0;
  if (t >= n_tiles) return;
  const GemmTile tile = load_tile(tiles, t);
  const bool on_diag = (tile.flags & kTileDiagonal) != 0;
  if (Q && on_diag && quarter == 2) return;      // below the diagonal: the mirror image of quarter 1
  const GemmProblem p = probs[tile.prob];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int fr = lane & 31, fh = lane >> 5;
  const int row0 = tile.r0 * kTileUnit + (Q ? 32 * (quarter >> 1) : 0), col0 = tile.c0 * kTileUnit + (Q ? 32 * (quarter & 1) : 0);
  const int slabs = p.K / BKF;                   // K is a multiple of 64
  // this wave's slabs: all of them, or wave, wave + 4, ...
  const int n = Q ? (slabs - wave + 3) / 4 : slabs;
  const int k_first = Q ? wave * BKF : 0, k_step = Q ? 4 * BKF : BKF;

  // ---- requests: a wave instruction fills 8 LDS rows; L rows first, then R rows.  Quarters: the wave's own 64 rows;
  // whole: instruction i of wave w fills rows 32 i + 8 w .. + 7 of the stage's 128.
  unsigned char* const my = smem + (Q ? wave * NST * 64 * ROWF : 0);
  constexpr int STAGE_B = Q ? 64 * ROWF : 128 * ROWF;
  const float* src[NLOAD];
#pragma unroll
  for (int i = 0; i < NLOAD; ++i) {
    const int r = (Q ? 8 * i : 32 * i + 8 * wave) + (lane >> 3);       // row of the stage
    const int chunk = (lane & 7) ^ ((r >> 1) & 7);
    src[i] = (r < ROWS ? static_cast<const float*>(p.L) + (size_t)(row0 + r) * p.ldl
                       : static_cast<const float*>(p.R) + (size_t)(col0 + r - ROWS) * p.ldr) + k_first + chunk * 4;
  }
  auto request = [&](int i_slab, int stage) {
    unsigned char* base = my + stage * STAGE_B + (Q ? 0 : wave * 1024);
    const size_t off = (size_t)i_slab * k_step;
#pragma unroll
    for (int i = 0; i < NLOAD; ++i)
      __builtin_amdgcn_global_load_lds((gptr)(src[i] + off), (lptr)(base + i * (Q ? 1024 : 4096)), 16, 0, 0);
  };

  // ---- fragments: lane (r = lane % 32, h = lane / 32) reads chunk 2 kk + h of its row, i.e. k = 8 kk + 4 h + 0..3; MFMA e
  // of a k-step multiplies k = 8 kk + e and 8 kk + 4 + e.
  const int fkey = (fr >> 1) & 7;
  const unsigned lds0 = (unsigned)(size_t)(lptr)my;
  const unsigned a_base = (unsigned)(((Q ? 0 : (wave >> 1) * 32) + fr) * ROWF);
  const unsigned b_base = (unsigned)((ROWS + (Q ? 0 : (wave & 1) * 32) + fr) * ROWF);
  HalfSlab half[2];
  auto read = [&](int stage, int which) {
    const unsigned s = lds0 + (unsigned)(stage * STAGE_B);
    const unsigned c0 = (unsigned)(((4 * which + fh) ^ fkey) * 16), c1 = (unsigned)(((4 * which + 2 + fh) ^ fkey) * 16);
    read_half(half[which], s + a_base + c0, s + a_base + c1, s + b_base + c0, s + b_base + c1);
  };
  // The order of a dot product's terms belongs to K alone, so that a matrix gets the same bits from whole entries and from
  // quarters, i.e. in any list: slab i goes to partial sum i % 4 (a quarter's wave holds one of the four, a whole entry's
  // wave all of them), and the result is (0 + 1) + (2 + 3).  LONG (K > 4096): an accumulator takes at most kFlush slabs
  // (512 terms) before it is added to its total, so the rounding error of a dot product grows with K / 2048 + 512 terms
  // instead of K / 4 (a single fp32 accumulator over 2^20 squares drifts by 4e-4 relative).
  // One accumulator per partial sum: MFMAs that wait for one another cost little beside the other waves' (16 of 512^2
  // 550 -> 556 us, 4 of 512^2 229 -> 224, 128 x 256 65.0 -> 64.2, against two that took turns in an order of each form's own);
  // two per partial sum spill in the whole form (602 us).  Chains that start at zero every slab, or every fourth, are more
  // exact beyond K = 512 (O of 1024^2 1.4e-6 -> 0.6e-6 and 1.0e-6) and cost 5 and 2 to 5 %.
  constexpr int kFlush = 16, NP = Q ? 1 : 4;
  f32x16 acc[NP], total[NP];
#pragma unroll
  for (int c = 0; c < NP; ++c)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[c][v] = total[c][v] = 0.f;
  auto flush = [&]() {
#pragma unroll
    for (int c = 0; c < NP; ++c)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        total[c][v] += acc[c][v];
        acc[c][v] = 0.f;
      }
  };
  auto mma = [&](const HalfSlab& f, auto c_tag) {
    constexpr int c = decltype(c_tag)::value;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[c] = __builtin_amdgcn_mfma_f32_32x32x2f32(f.a[kk][e], f.b[kk][e], acc[c], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  };

#pragma unroll
  for (int s = 0; s < NST; ++s)
    if (s < n) request(s, s);
  float alpha = 1.f;
  if (Q && alpha_idx == kAlphaFromPartials) {
    // first Gram product: the norm, from the partial sums
    float s, s2;
    norm_scalars(block_sum_f64(p.partials, p.n_part, reinterpret_cast<double*>(smem + lds_bytes(true))), eps, &s, &s2);
    if (row0 == 0 && col0 == 0 && tid == 0) {
      float* scal = const_cast<float*>(p.scal);
      scal[0] = s;
      scal[1] = s2;
    }
    alpha = s2;
  } else if (alpha_idx >= 0) {
    alpha = p.scal[alpha_idx];
  }
  if (n > 0) {
    if (!Q && n >= 3) wait_vmcnt<2 * NLOAD>();
    else if (n >= 2) wait_vmcnt<NLOAD>();
    else wait_vmcnt<0>();
    if (!Q) __builtin_amdgcn_s_barrier();
    read(0, 0);
    land_half(half[0]);
    int stage = 0;
    // slab i with others behind it, and the last one.  The first half is landed where the slab begins: a read in flight
    // must not cross a branch, where the compiler may move its registers.
    auto slab = [&](int i, auto c_tag) {
      read(stage, 1);
      mma(half[0], c_tag);
      land_half(half[1]);
      const int next = stage + 1 == NST ? 0 : stage + 1;
      if (Q) {
        // the stage is this wave's own and has been read: refill it, then wait for the next slab
        if (i + NST < n) request(i + NST, stage);
        if (i + 2 < n) wait_vmcnt<NLOAD>();
        else wait_vmcnt<0>();
      } else {
        if (i + 2 < n) wait_vmcnt<NLOAD>();      // my requests of the next slab have landed (one slab is behind it)
        else wait_vmcnt<0>();
        __builtin_amdgcn_s_barrier();            // everybody's; and everybody has read this one: its stage is refilled
        if (i + NST < n) request(i + NST, stage);
      }
      read(next, 0);
      mma(half[1], c_tag);
      land_half(half[0]);
      stage = next;
    };
    auto last_slab = [&](auto c_tag) {
      read(stage, 1);
      mma(half[0], c_tag);
      land_half(half[1]);
      mma(half[1], c_tag);
    };
    using P0 = std::integral_constant<int, 0>;
    using P1 = std::integral_constant<int, Q ? 0 : 1>;
    using P2 = std::integral_constant<int, Q ? 0 : 2>;
    using P3 = std::integral_constant<int, Q ? 0 : 3>;
    int i = 0, since = 0;
    if constexpr (Q) {
      for (; i + 1 < n; ++i) {
        slab(i, P0{});
        if (LONG && ++since == kFlush) {
          since = 0;
          flush();
        }
      }
      last_slab(P0{});
    } else {                                     // n is even
      for (; i + 4 < n; i += 4) {
        slab(i, P0{});
        slab(i + 1, P1{});
        slab(i + 2, P2{});
        slab(i + 3, P3{});
        if (LONG && ++since == kFlush) {
          since = 0;
          flush();
        }
      }
      slab(i, P0{});
      if (n - i == 2) {
        last_slab(P1{});
      } else {
        slab(i + 1, P1{});
        slab(i + 2, P2{});
        last_slab(P3{});
      }
    }
  }
  if constexpr (LONG) flush();
  f32x16 sum = LONG ? total[0] : acc[0];         // quarters: this wave's partial sum, added to the others' below
  if constexpr (!Q) {
    const f32x16 *const t = LONG ? total : acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) sum[v] = (t[0][v] + t[1][v]) + (t[2][v] + t[3][v]);
  }

  // ---- epilogue.  A lane holds column fr, rows 8 q + 4 h + e of its wave's 32 x 32 tile: it goes to LDS as image
  // [column][row].  Quarters: the four waves' partial tiles are added up, one float4 per thread; whole: each wave reads
  // its own tile back.  Et is the addend stored transposed, so that it is read and Ct written along rows of the image.
  float* C = static_cast<float*>(p.C);
  float* Ct = static_cast<float*>(p.Ct);
  int ldct = p.ldct;
  if (p.symmetric) {                             // mirror store; the tile itself only on the diagonal
    Ct = on_diag && (!Q || quarter != 1) ? nullptr : C;
    ldct = p.ldc;
  }
  // The addend, this thread's float4s of the transposed tile: whole entries ask for it before the block meets and the tile
  // passes through the LDS (-1 to -2 % of a step); in quarters, one float4 behind a longer sum, that place gains nothing.
  constexpr int NV = Q ? 1 : 4;                  // float4s per thread
  const float* Et = static_cast<const float*>(p.Et);
  const int sub_r = Q ? 0 : (wave >> 1) * 32, sub_c = Q ? 0 : (wave & 1) * 32;
  f32x4 ev[NV];
  auto load_e = [&](int u) {
    const int c = Q ? tid >> 3 : (lane >> 3) + 8 * u, r4 = 4 * (lane & 7);
    ev[u] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (Et) ev[u] = *reinterpret_cast<const f32x4*>(Et + (size_t)(col0 + sub_c + c) * p.ldet + row0 + sub_r + r4);
  };
  if constexpr (!Q) {
#pragma unroll
    for (int u = 0; u < NV; ++u) load_e(u);
  }
  meet();                                        // every wave is done with the ring
  float* const img = reinterpret_cast<float*>(smem) + wave * 32 * kImgPitch;
#pragma unroll
  for (int q = 0; q < 4; ++q)
    *reinterpret_cast<f32x4*>(img + fr * kImgPitch + 8 * q + 4 * fh) = f32x4{sum[4 * q], sum[4 * q + 1], sum[4 * q + 2], sum[4 * q + 3]};
  meet();
  f32x4 val[NV];
#pragma unroll
  for (int u = 0; u < NV; ++u) {
    const int c = Q ? tid >> 3 : (lane >> 3) + 8 * u, r4 = 4 * (lane & 7);
    f32x4 x;
    if (Q) {
      const float* s0 = reinterpret_cast<const float*>(smem) + c * kImgPitch + r4;
      const f32x4 x0 = *reinterpret_cast<const f32x4*>(s0), x1 = *reinterpret_cast<const f32x4*>(s0 + 32 * kImgPitch);
      const f32x4 x2 = *reinterpret_cast<const f32x4*>(s0 + 64 * kImgPitch), x3 = *reinterpret_cast<const f32x4*>(s0 + 96 * kImgPitch);
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = (x0[e] + x1[e]) + (x2[e] + x3[e]);
    } else {
      x = *reinterpret_cast<const f32x4*>(img + c * kImgPitch + r4);
    }
    if constexpr (Q) load_e(u);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float y = beta_acc * x[e];
      if (Et) y = fmaf(beta_e, ev[u][e], y);
      val[u][e] = alpha * y;
    }
    if (Ct) *reinterpret_cast<f32x4*>(Ct + (size_t)(col0 + sub_c + c) * ldct + row0 + sub_r + r4) = val[u];
  }
  if (C) {
    __syncthreads();                             // the image has been read: it takes the results as [row][column]
    float* const out = Q ? reinterpret_cast<float*>(smem) : img;
#pragma unroll
    for (int u = 0; u < NV; ++u) {
      const int c = Q ? tid >> 3 : (lane >> 3) + 8 * u, r4 = 4 * (lane & 7);
#pragma unroll
      for (int e = 0; e < 4; ++e) out[(r4 + e) * kImgPitch + c] = val[u][e];
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < NV; ++u) {
      const int r = Q ? tid >> 3 : (lane >> 3) + 8 * u, c4 = 4 * (lane & 7);
      *reinterpret_cast<f32x4*>(C + (size_t)(row0 + sub_r + r) * p.ldc + col0 + sub_c + c4) =
          *reinterpret_cast<const f32x4*>(out + r * kImgPitch + c4);
    }
  }
}

template <bool LONG>
hipError_t setup_f32() {
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&ns_gemm_f32_kernel<true, LONG>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)(lds_bytes(true) + kLdsFold));
  if (e != hipSuccess) return e;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&ns_gemm_f32_kernel<false, LONG>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes(false));
}

template <bool LONG>
void launch_f32(int flags, int tail, const GemmProblem* probs, const GemmTile* tiles, int n_tiles, float beta_acc, float beta_e, int alpha_idx,
                double eps, hipStream_t s) {
  if (flags & kGemmQuarters)
    ns_gemm_f32_kernel<true, LONG><<<(n_tiles + 7) / 8 * 32, 256, lds_bytes(true) + (alpha_idx == kAlphaFromPartials ? kLdsFold : 0), s>>>(
        probs, tiles, n_tiles, beta_acc, beta_e, alpha_idx, eps);
  else {
    ns_gemm_f32_kernel<false, LONG><<<n_tiles - tail, 256, lds_bytes(false), s>>>(probs, tiles, n_tiles - tail, beta_acc, beta_e, alpha_idx, eps);
    if (tail > 0)
      ns_gemm_f32_kernel<true, LONG><<<(tail + 7) / 8 * 32, 256, lds_bytes(true), s>>>(probs, tiles + (n_tiles - tail), tail, beta_acc, beta_e,
                                                                                       alpha_idx, eps);
  }
}

}  // namespace

hipError_t gemm_f32_setup() {
  const hipError_t e = setup_f32<false>();
  return e != hipSuccess ? e : setup_f32<true>();
}

hipError_t launch_gemm_f32(int flags, int tail, const GemmProblem* probs, const GemmTile* tiles, int n_tiles, float beta_acc, float beta_e,
                           int alpha_idx, double eps, hipStream_t s) {
  if (n_tiles <= 0) return hipSuccess;
  if (tail < 0 || tail >= n_tiles) return hipErrorInvalidValue;
  if (alpha_idx == kAlphaFromPartials && !(flags & kGemmQuarters)) return hipErrorInvalidValue;
  if (flags & kGemmLongK) launch_f32<true>(flags, tail, probs, tiles, n_tiles, beta_acc, beta_e, alpha_idx, eps, s);
  else launch_f32<false>(flags, tail, probs, tiles, n_tiles, beta_acc, beta_e, alpha_idx, eps, s);
  return hipGetLastError();
}

}  // namespace muon
