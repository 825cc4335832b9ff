// HBM-bound kernels of the Muon step for gfx950: momentum + Frobenius partials + cast/orient,
// norm finalisation, the scaled weight-decayed apply, update-RMS and a test read-back.
//
// All of them walk a table of 64x64 element tiles so that one launch covers every matrix of a chunk.
#include <hip/hip_runtime.h>

#include "muon_launch.h"

namespace muon {
namespace {

typedef unsigned short u16;

__device__ __forceinline__ float bf16_to_f32(u16 h) { return __uint_as_float(((unsigned)h) << 16); }

// round-to-nearest-even, NaN kept quiet
__device__ __forceinline__ u16 f32_to_bf16(float f) {
  unsigned u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (u16)((u >> 16) | 0x40u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (u16)(u >> 16);
}

typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

// two floats -> packed bf16 pair, round-to-nearest-even (one v_cvt_pk_bf16_f32)
__device__ __forceinline__ unsigned pack2(float lo, float hi) {
  const f32x2_t v = {lo, hi};
  return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2_t));
}

// Deterministic block-wide sum (256 threads): butterfly inside each wave, then the 4 wave sums in order.
__device__ __forceinline__ float block_sum_256(float v, float* red /* >= 4 floats of LDS */) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) red[wave] = v;
  __syncthreads();
  return (red[0] + red[1]) + (red[2] + red[3]);
}

// Value of lane S of this lane's group of four.
template <int S>
__device__ __forceinline__ float quad_lane(float v) {
  constexpr int ctrl = S | (S << 2) | (S << 4) | (S << 6);
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), ctrl, 0xf, 0xf, true));
}

// Value of the lane N places on, around this lane's group of sixteen.
template <int N>
__device__ __forceinline__ float row_rotate(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + N, 0xf, 0xf, true));
}

// Sum of squares of a 64 x 64 tile of which thread t holds columns 4 (t % 16) .. + 3 of rows t / 16 + 16 j, in an order that
// belongs to the tile and not to this distribution: 16 consecutive columns of a row are one chain of fma; the 64 chains of
// 16 consecutive rows (chain 4 (r % 16) + c / 16) are added up as a tree (32 apart first, neighbours last); the four
// results as (0 + 1) + (2 + 3).  The last bits of the norm decide bf16 roundings of everything behind it, so another
// order would be another result (up to 6e-4 of the updated weights).  A chain passes through the four lanes that hold
// its columns.  Contains one barrier; the sum is valid in the first wave.
// Against sums of each thread's own elements: 0.2 us on a launch of a few blocks, nothing on long lists, which memory bounds.
__device__ __forceinline__ float tile_sum_squares(const float (&u)[4][4], float* red /* 256 floats of LDS */) {
  const int tid = threadIdx.x;
  auto chain = [](float c, const float (&x)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) c = fmaf(x[i], x[i], c);
    return c;
  };
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    float c = chain(0.f, u[j]);                  // right in the first lane of four, then in the second, ...
    c = chain(quad_lane<0>(c), u[j]);
    c = chain(quad_lane<1>(c), u[j]);
    c = chain(quad_lane<2>(c), u[j]);
    if ((tid & 3) == 3) red[64 * j + (tid >> 2)] = c;
  }
  __syncthreads();
  float t = 0.f;
  if (tid < 64) {
    const float* v = red + 64 * (tid >> 4) + (tid & 15);       // 16 lanes for each group of 64 chains
    t = (v[0] + v[32]) + (v[16] + v[48]);
    t += row_rotate<8>(t);                       // t repeats every 8 lanes now, then every 4, ...: a rotation is the exchange
    t += row_rotate<4>(t);
    t += row_rotate<2>(t);
    t += row_rotate<1>(t);
    auto lane = [&](int l) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(t), l)); };
    t = (lane(0) + lane(16)) + (lane(32) + lane(48));
  }
  return t;
}

// Accesses go through the global address space (pointers that come out of a table would otherwise be accessed as
// `flat`).  Those to the caller's matrices are wide at any alignment of the element: rows start anywhere, and global
// memory takes such accesses (the vector types only tell the compiler), so odd widths and odd buffers keep the wide path.
#define MUON_GLOBAL __attribute__((address_space(1)))
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned int u32x4_any __attribute__((ext_vector_type(4), aligned(2)));
typedef unsigned int u32x2_any __attribute__((ext_vector_type(2), aligned(2)));

// 4 consecutive elements
__device__ __forceinline__ void load4(const float* p, float* out) {
  const f32x4_any v = *(const MUON_GLOBAL f32x4_any*)p;
#pragma unroll
  for (int i = 0; i < 4; ++i) out[i] = v[i];
}
__device__ __forceinline__ void load4(const u16* p, float* out) {
  const u32x2_any v = *(const MUON_GLOBAL u32x2_any*)p;
  out[0] = __uint_as_float(v.x << 16);
  out[1] = __uint_as_float(v.x & 0xffff0000u);
  out[2] = __uint_as_float(v.y << 16);
  out[3] = __uint_as_float(v.y & 0xffff0000u);
}
__device__ __forceinline__ void store4(float* p, const float* in) { *(MUON_GLOBAL f32x4_any*)p = f32x4_any{in[0], in[1], in[2], in[3]}; }
__device__ __forceinline__ void store4(u16* p, const float* in) {
  *(MUON_GLOBAL u32x2_any*)p = u32x2_any{pack2(in[0], in[1]), pack2(in[2], in[3])};
}

template <typename T>
__device__ __forceinline__ float load1(const T* p);
template <>
__device__ __forceinline__ float load1<float>(const float* p) { return *(const MUON_GLOBAL float*)p; }
template <>
__device__ __forceinline__ float load1<u16>(const u16* p) { return bf16_to_f32(*(const MUON_GLOBAL u16*)p); }
template <typename T>
__device__ __forceinline__ void store1(T* p, float v);
template <>
__device__ __forceinline__ void store1<float>(float* p, float v) { *(MUON_GLOBAL float*)p = v; }
template <>
__device__ __forceinline__ void store1<u16>(u16* p, float v) { *(MUON_GLOBAL u16*)p = f32_to_bf16(v); }

// Newton-Schulz storage with PL planes (PL = 1: one array of XT; PL > 1, XT = bf16: the value is the sum of PL bf16
// arrays `plane` elements apart, array q holding what the arrays before it left of the fp32 value after rounding).
template <typename XT, int PL>
__device__ __forceinline__ void ns_store4(XT* p, size_t plane, const float* in) {
  if constexpr (PL == 1) {
    store4(p, in);
  } else {
    float rest[4] = {in[0], in[1], in[2], in[3]};
#pragma unroll
    for (int q = 0; q < PL; ++q) {
      store4(p + q * plane, rest);
      if (q + 1 < PL) {
#pragma unroll
        for (int i = 0; i < 4; i += 2) {
          const unsigned w = pack2(rest[i], rest[i + 1]);
          rest[i] -= __uint_as_float(w << 16);              // exact: the rounding error of an fp32 value is an fp32 value
          rest[i + 1] -= __uint_as_float(w & 0xffff0000u);
        }
      }
    }
  }
}
template <typename XT, int PL>
__device__ __forceinline__ float ns_load1(const XT* p, size_t plane) {
  float v = load1<XT>(p + (PL - 1) * plane);
  if constexpr (PL > 1) {
#pragma unroll
    for (int q = PL - 2; q >= 0; --q) v += load1<XT>(p + q * plane);
  }
  return v;
}

// ------------------------------------------------------------------------------------------------------
// a1 + a2 (first stage) + a3.  Thread t of a block owns columns 4 (t % 16) .. + 3 of rows t / 16 + 16 j, j = 0..3, of a
// 64x64 tile in U's orientation: the 16 lanes that share a row cover whole lines with every access.  GT: gradient element
// type; XT: Newton-Schulz element type.
// Writes: M (guarded), the tile of U into the buffer of the same orientation, the transposed tile (through
// LDS) into the buffer of the other orientation, both zero-filled outside A x B, and one partial sum of U^2.
// Bound by memory on long lists (4 of 4096^2: 152 -> 136 us, 5.9 TB/s of its 12 B per element, when the lanes of a row took
// 16 consecutive elements each), by the latency of one chain of loads on short ones.  Rows of any width take the wide path:
// 50 of 2047 x 1401 3074 -> 404 us, six matrices of odd widths 106 -> 32 us, against scalar accesses whose loads waited
// for the stores before them.  Non-temporal hints: -4 % on aligned rows, +40 % on odd ones, not used.
// ------------------------------------------------------------------------------------------------------
template <typename GT, typename XT, int PL>
__device__ __forceinline__ void momentum_tile(const MatDesc& d, const MatPtrs& pt, int tr, int tc, float mu, int nesterov,
                                              bool both, float (*lds)[kEwTile + 1], float* red) {
  const int tid = threadIdx.x;
  const int lr = tid >> 4, lc = (tid & 15) * 4;
  const int r0 = tr * kEwTile + lr, c0 = tc * kEwTile + lc;
  const int A = d.rows, B = d.cols;
  const GT* g = static_cast<const GT*>(pt.g);
  float* m = pt.m;

  float u[4][4], mv[4][4], gv[4][4];
  const bool wide = c0 + 4 <= B;
  // all loads are issued before the first store
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int r = r0 + 16 * j;
    const size_t base = (size_t)r * (size_t)B + (size_t)c0;
    if (wide && r < A) {
      load4(m + base, mv[j]);
      load4(g + base, gv[j]);
    } else {                                     // the right edge, or beyond the matrix
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bool in = r < A && c0 + i < B;
        mv[j][i] = in ? load1<float>(m + base + i) : 0.f;
        gv[j][i] = in ? load1<GT>(g + base + i) : 0.f;
      }
    }
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int r = r0 + 16 * j;
    const size_t base = (size_t)r * (size_t)B + (size_t)c0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float mn = fmaf(mu, mv[j][i], gv[j][i]);
      mv[j][i] = mn;
      u[j][i] = nesterov ? fmaf(mu, mn, gv[j][i]) : mn;
    }
    if (wide && r < A) {
      store4(m + base, mv[j]);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (r < A && c0 + i < B) store1<float>(m + base + i, mv[j][i]);
    }
  }

  // Orientation: the buffer whose rows run along U's rows, and the one holding U^T.
  // not transposed: X = U (pitch np), Xt = U^T (pitch mp).  transposed: Xt = U (pitch mp), X = U^T (pitch np).
  XT* same = static_cast<XT*>(d.transposed ? d.Xt[0] : d.X);
  XT* flip = static_cast<XT*>(d.transposed ? d.X : d.Xt[0]);
  const int pitch_same = d.transposed ? d.mp : d.np;
  const int pitch_flip = d.transposed ? d.np : d.mp;

  const bool write_same = both || !d.transposed, write_flip = both || d.transposed;
  if (write_same) {
#pragma unroll
    for (int j = 0; j < 4; ++j) ns_store4<XT, PL>(same + (size_t)(r0 + 16 * j) * pitch_same + c0, (size_t)d.x_plane, u[j]);
  }

  // the transposed tile goes through LDS; skipped (block-uniformly) where only the untransposed layout is wanted
  if (write_flip) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i) lds[lc + i][lr + 16 * j] = u[j][i];
  }
  const float total = tile_sum_squares(u, red);   // contains the barrier that publishes the LDS tile
  if (write_flip) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int fc = lr + 16 * j;                // row of U^T (= column of U), 4 consecutive columns of U^T
      float t[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) t[i] = lds[fc][lc + i];
      ns_store4<XT, PL>(flip + (size_t)(tc * kEwTile + fc) * pitch_flip + tr * kEwTile + lc, (size_t)d.x_plane, t);
    }
  }

  if (tid == 0) d.partials[tr * d.ew_tiles_c + tc] = total;
}

// A block's work item through whole-dword loads, so that they are scalar loads (uniform address).
__device__ __forceinline__ EwTile load_item(const EwTile* __restrict__ tiles) {
  static_assert(sizeof(EwTile) == 12, "three dwords");
  const uint32_t* w = reinterpret_cast<const uint32_t*>(tiles) + 3 * (size_t)blockIdx.x;
  const uint32_t w0 = w[0], w1 = w[1], w2 = w[2];
  EwTile t;
  t.mat = (int32_t)w0;
  t.tr = (int16_t)(w1 & 0xffffu);
  t.tc = (int16_t)(w1 >> 16);
  t.count = (int16_t)(w2 & 0xffffu);
  t.pad_ = 0;
  return t;
}

template <typename XT, int PL>
__device__ __forceinline__ void momentum_item(const MatDesc& d, const MatPtrs& pt, const EwTile& t, float mu, int nesterov, int both) {
  __shared__ float lds[kEwTile][kEwTile + 1];
  __shared__ float red[256];
  for (int k = 0; k < t.count; ++k) {
    if (k) __syncthreads();     // the LDS tile and the reduction scratch are reused
    if (d.g_dtype == kDtypeBF16)
      momentum_tile<u16, XT, PL>(d, pt, t.tr, t.tc + k, mu, nesterov, both != 0, lds, red);
    else
      momentum_tile<float, XT, PL>(d, pt, t.tr, t.tc + k, mu, nesterov, both != 0, lds, red);
  }
}

template <typename XT, int PL>
__global__ __launch_bounds__(256) void momentum_norm_cast_kernel(const MatDesc* __restrict__ mats,
                                                                  const MatPtrs* __restrict__ ptrs,
                                                                  const EwTile* __restrict__ tiles, float mu,
                                                                  int nesterov, int both) {
  const EwTile t = load_item(tiles);
  const MatDesc& d = mats[t.mat];     // read in place (uniform address: scalar loads); see o_source
  const MatPtrs pt = ptrs[t.mat];
  momentum_item<XT, PL>(d, pt, t, mu, nesterov, both);
}

// The same with the step's pointers as a kernel argument; a matrix's first block leaves them in the table for the passes
// behind this one (a launch of its own for the table cost 3 us).
template <typename XT, int PL>
__global__ __launch_bounds__(256) void momentum_norm_cast_pack_kernel(const MatDesc* __restrict__ mats, PtrPack pack,
                                                                       MatPtrs* __restrict__ ptrs,
                                                                       const EwTile* __restrict__ tiles, float mu,
                                                                       int nesterov, int both) {
  const EwTile t = load_item(tiles);
  const MatDesc& d = mats[t.mat];
  const MatPtrs pt = pack.p[t.mat];
  if (t.tr == 0 && t.tc == 0 && threadIdx.x == 0) ptrs[t.mat] = pt;
  momentum_item<XT, PL>(d, pt, t, mu, nesterov, both);
}

// ------------------------------------------------------------------------------------------------------
// a2 second stage: one block per matrix sums its partials in a fixed order, in double.
// ------------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void norm_finalize_kernel(const MatDesc* __restrict__ mats, int first_mat, double eps, float gram_gain) {
  __shared__ double red[256];
  const MatDesc& d = mats[first_mat + blockIdx.x];
  const double sum = block_sum_f64(d.partials, d.n_part, red);
  if (threadIdx.x == 0) {
    float s, s2;
    norm_scalars(sum, eps, &s, &s2);
    store_norm(d.scal, sum, eps, d.gram_route ? gram_gain : 0.f, s, s2);
  }
}

// ------------------------------------------------------------------------------------------------------
// a8: W <- W - lr * (rms_scale*sqrt(max(A,B)) * O + wd * W), fp32 math, one rounding to W's dtype.
// ------------------------------------------------------------------------------------------------------
// Where O (in W's orientation) lives after the Newton-Schulz phase.  o_sel bit 0: which of Xt[0..1] for matrices
// iterated on their transpose; bit 1: X (0) or Xt[0] used as the second m_pad x n_pad buffer (1) for the others.
// The record is read in place, never copied into a local: with a local copy the compiler turned the selections below
// into loads from a selected address of that copy, which put the whole 128-byte record into per-thread scratch memory
// - 8 bytes of scratch traffic per matrix element; the HBM-side write counter of the update kernel read twice the
// bytes of W because of it.
// Bits 2 and 3: the same for matrices of the Gram route, whose iterate changes buffers once per group of iterations.
__device__ __forceinline__ const void* o_source(const MatDesc& d, int o_sel) {
  if (d.gram_route) o_sel >>= 2;
  if (d.transposed) return (o_sel & 1) ? d.Xt[1] : d.Xt[0];
  return (o_sel & 2) ? d.Xt[0] : d.X;
}

// 8 consecutive elements at element alignment: one 16-byte access for bf16, two for fp32.  Streaming hint on bf16: every
// element of the update is touched once; without it the L2 refetched a third of the lines (measured: 1.20 GB fetched for
// 0.81 GB of W and O on the 4096-wide block, 0.89 GB with the hint).  The hint leaves more of the caches to the next step's
// momentum pass (50 of 2048 x 1408: update 164 us with it, 160 without, momentum 319 and 343).  Long lists whose
// rows do not end on whole lines take W without it (STREAM = false): a line written in two pieces leaves the caches between
// them.  Step of 50 of 2047 x 1401 4881 us with the hint on W, 4700 without, of 2048 x 1400 4806 / 4676.  (Kernels of their own: with
// both bodies in one and the hint as an argument short lists' updates took 0.7 us longer, 43 of up to 3840 columns 8.3 / 9.0.)
template <bool STREAM = true>
__device__ __forceinline__ void load8(const float* p, float* out) {
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const f32x4_any v = ((const MUON_GLOBAL f32x4_any*)p)[i];
    out[4 * i + 0] = v.x; out[4 * i + 1] = v.y; out[4 * i + 2] = v.z; out[4 * i + 3] = v.w;
  }
}
template <bool STREAM = true>
__device__ __forceinline__ void load8(const u16* p, float* out) {
  u32x4_any v;
  if constexpr (STREAM) v = __builtin_nontemporal_load((const MUON_GLOBAL u32x4_any*)p);
  else v = *(const MUON_GLOBAL u32x4_any*)p;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    out[2 * j] = __uint_as_float(v[j] << 16);
    out[2 * j + 1] = __uint_as_float(v[j] & 0xffff0000u);
  }
}
template <bool STREAM>
__device__ __forceinline__ void store8(float* p, const float* in) {
#pragma unroll
  for (int i = 0; i < 2; ++i) ((MUON_GLOBAL f32x4_any*)p)[i] = f32x4_any{in[4 * i], in[4 * i + 1], in[4 * i + 2], in[4 * i + 3]};
}
template <bool STREAM>
__device__ __forceinline__ void store8(u16* p, const float* in) {
  const u32x4_any v = {pack2(in[0], in[1]), pack2(in[2], in[3]), pack2(in[4], in[5]), pack2(in[6], in[7])};
  if constexpr (STREAM) __builtin_nontemporal_store(v, (MUON_GLOBAL u32x4_any*)p);
  else *(MUON_GLOBAL u32x4_any*)p = v;
}
template <typename XT, int PL>
__device__ __forceinline__ void ns_load8(const XT* p, size_t plane, float* out) {
  load8(p + (PL - 1) * plane, out);
  if constexpr (PL > 1) {
#pragma unroll
    for (int q = PL - 2; q >= 0; --q) {        // smallest plane first
      float v[8];
      load8(p + q * plane, v);
#pragma unroll
      for (int i = 0; i < 8; ++i) out[i] += v[i];
    }
  }
}

// One 64x64 tile of the update.  Thread t owns 8 consecutive columns, (t % 8) * 8 .., of rows t / 8 and t / 8 + 32:
// the 8 lanes that share a row cover one whole 128-byte line of a bf16 array with every load or store instruction
// (a thread that owned 16 consecutive elements wrote every line in two instructions of scattered 16-byte pieces).
template <typename WT, typename XT, int PL, bool UPDATE, bool STREAM>
__device__ __forceinline__ void apply_tile(const MatDesc& d, const MatPtrs& pt, int tr, int tc, float lr, float wd,
                                           float scale, int o_sel, float* red) {
  const int tid = threadIdx.x;
  const int c0 = tc * kEwTile + (tid & 7) * 8;
  const int A = d.rows, B = d.cols;
  WT* w = static_cast<WT*>(pt.w);
  const XT* o = static_cast<const XT*>(o_source(d, o_sel));
  const int pitch = d.transposed ? d.mp : d.np;
  const size_t plane = (size_t)d.x_plane;
  const int r0 = tr * kEwTile + (tid >> 3), r1 = r0 + 32;
  float ss = 0.f;
  const bool wide = c0 + 8 <= B;
  if (wide && r1 < A) {
    // both rows at once: all loads are issued before the first store
    float ov[2][8], wv[2][8];
    ns_load8<XT, PL>(o + (size_t)r0 * pitch + c0, plane, ov[0]);
    ns_load8<XT, PL>(o + (size_t)r1 * pitch + c0, plane, ov[1]);
    if (UPDATE) {
      load8<STREAM>(w + (size_t)r0 * (size_t)B + c0, wv[0]);
      load8<STREAM>(w + (size_t)r1 * (size_t)B + c0, wv[1]);
    }
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        ss = fmaf(ov[u][i], ov[u][i], ss);
        if (UPDATE) {
          const float t = fmaf(wd, wv[u][i], scale * ov[u][i]);
          wv[u][i] = fmaf(-lr, t, wv[u][i]);
        }
      }
    if (UPDATE) {
      store8<STREAM>(w + (size_t)r0 * (size_t)B + c0, wv[0]);
      store8<STREAM>(w + (size_t)r1 * (size_t)B + c0, wv[1]);
    }
  } else if (c0 < B) {
    // the matrix's bottom rows, which stay wide, and its right edge.  O's columns are padded to whole tiles, so it is read
    // wide everywhere; rows beyond the matrix are not read (64 of 16 x 4096: 12 us; 22 with them, 27 with W one element
    // at a time as well).  The elements of W are all loaded before the first one is stored.
    float ov[2][8], wv[2][8];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int r = u ? r1 : r0;
      if (r >= A) continue;
      ns_load8<XT, PL>(o + (size_t)r * pitch + c0, plane, ov[u]);
      if (UPDATE && wide) {
        load8<STREAM>(w + (size_t)r * (size_t)B + c0, wv[u]);
      } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) wv[u][i] = UPDATE && c0 + i < B ? load1<WT>(w + (size_t)r * (size_t)B + c0 + i) : 0.f;
      }
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int r = u ? r1 : r0;
      if (r >= A) continue;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        ss = c0 + i < B ? fmaf(ov[u][i], ov[u][i], ss) : ss;
        if (UPDATE) {
          const float t = fmaf(wd, wv[u][i], scale * ov[u][i]);
          wv[u][i] = fmaf(-lr, t, wv[u][i]);
        }
      }
      if (UPDATE && wide) {
        store8<STREAM>(w + (size_t)r * (size_t)B + c0, wv[u]);
      } else if (UPDATE) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
          if (c0 + i < B) store1<WT>(w + (size_t)r * (size_t)B + c0 + i, wv[u][i]);
      }
    }
  }
  const float total = block_sum_256(ss, red);
  if (tid == 0) d.partials[tr * d.ew_tiles_c + tc] = total;
}

template <typename XT, int PL, bool STREAM>
__global__ __launch_bounds__(256) void apply_update_kernel(const MatDesc* __restrict__ mats, const MatPtrs* __restrict__ ptrs,
                                                            const EwTile* __restrict__ tiles, float lr, float wd,
                                                            float rms_scale, int scale_mode, float sqrt_hidden, int o_sel,
                                                            int use_s) {
  __shared__ float red[4];
  const EwTile t = load_item(tiles);
  const MatDesc& d = mats[t.mat];       // read in place (uniform address: scalar loads); see o_source
  const MatPtrs pt = ptrs[t.mat];
  // factor that multiplies the stored O: the three variants of section 3.1 (Eq. 5-7)
  float scale;
  if (scale_mode == 2) {
    scale = rms_scale * d.scal[2];              // 1/RMS of the stored O: any common factor of O cancels
  } else {
    scale = rms_scale * (scale_mode == 1 ? sqrt_hidden : d.sqrt_max);
    if (use_s) scale *= d.scal[0];
  }
  for (int k = 0; k < t.count; ++k) {
    if (k) __syncthreads();     // the reduction scratch is reused
    if (d.w_dtype == kDtypeBF16)
      apply_tile<u16, XT, PL, true, STREAM>(d, pt, t.tr, t.tc + k, lr, wd, scale, o_sel, red);
    else
      apply_tile<float, XT, PL, true, STREAM>(d, pt, t.tr, t.tc + k, lr, wd, scale, o_sel, red);
  }
}

// Per-tile sums of O^2 only (first pass of the "Update Norm" variant, Eq. 6).
template <typename XT, int PL>
__global__ __launch_bounds__(256) void update_sumsq_kernel(const MatDesc* __restrict__ mats, const EwTile* __restrict__ tiles,
                                                            int o_sel) {
  __shared__ float red[4];
  const EwTile t = load_item(tiles);
  const MatDesc& d = mats[t.mat];       // read in place (uniform address: scalar loads); see o_source
  const MatPtrs none{nullptr, nullptr, nullptr};
  for (int k = 0; k < t.count; ++k) {
    if (k) __syncthreads();
    apply_tile<float, XT, PL, false, true>(d, none, t.tr, t.tc + k, 0.f, 0.f, 0.f, o_sel, red);
  }
}

// sqrt(mean(O^2)) per matrix from the per-tile sums left by apply_update_kernel.
__global__ __launch_bounds__(256) void update_rms_kernel(const MatDesc* __restrict__ mats, int first_mat, int use_s,
                                                          int to_scal, float* __restrict__ out) {
  __shared__ double red[256];
  const MatDesc& d = mats[first_mat + blockIdx.x];
  const double sum = block_sum_f64(d.partials, d.n_part, red);
  if (threadIdx.x == 0) {
    double rms = sqrt(sum / ((double)d.rows * (double)d.cols));
    if (to_scal) {
      d.scal[2] = rms > 0.0 ? (float)(1.0 / rms) : 0.f;
    } else {
      if (use_s) rms *= (double)d.scal[0];
      out[first_mat + blockIdx.x] = (float)rms;
    }
  }
}

template <typename XT, int PL, typename DT>
__global__ __launch_bounds__(256) void read_update_kernel(const MatDesc* __restrict__ mats, int mat, int o_sel, int use_s,
                                                           DT* __restrict__ dst) {
  const MatDesc& d = mats[mat];
  const XT* o = static_cast<const XT*>(o_source(d, o_sel));
  const int pitch = d.transposed ? d.mp : d.np;
  const float s = use_s ? d.scal[0] : 1.f;
  const size_t total = (size_t)d.rows * (size_t)d.cols;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (size_t)gridDim.x * 256) {
    const size_t r = i / (size_t)d.cols, c = i % (size_t)d.cols;
    store1<DT>(dst + i, s * ns_load1<XT, PL>(o + r * pitch + c, (size_t)d.x_plane));
  }
}

}  // namespace

// ns_dtype -> (element type, planes): fp32; bf16; bf16 x 2 planes; bf16 x 3 planes
#define MUON_NS_DISPATCH(ns_dtype, CALL)                 \
  switch (ns_dtype) {                                    \
    case kDtypeF32: { CALL(float, 1); break; }           \
    case kDtypeBF16: { CALL(u16, 1); break; }            \
    case kDtypeBF16X2: { CALL(u16, 2); break; }          \
    case kDtypeBF16X3: { CALL(u16, 3); break; }          \
    default: return hipErrorInvalidValue;                \
  }

hipError_t launch_momentum_norm_cast(const MatDesc* mats, MatPtrs* ptrs, const PtrPack* pack, const EwTile* tiles, int n_tiles,
                                     float mu, int nesterov, int both_layouts, int ns_dtype, hipStream_t s) {
  if (n_tiles <= 0) return hipSuccess;
  if (pack) {
#define MUON_CALL(XT, PL) \
  momentum_norm_cast_pack_kernel<XT, PL><<<n_tiles, 256, 0, s>>>(mats, *pack, ptrs, tiles, mu, nesterov, both_layouts)
    MUON_NS_DISPATCH(ns_dtype, MUON_CALL)
#undef MUON_CALL
  } else {
#define MUON_CALL(XT, PL) momentum_norm_cast_kernel<XT, PL><<<n_tiles, 256, 0, s>>>(mats, ptrs, tiles, mu, nesterov, both_layouts)
    MUON_NS_DISPATCH(ns_dtype, MUON_CALL)
#undef MUON_CALL
  }
  return hipGetLastError();
}

hipError_t launch_norm_finalize(const MatDesc* mats, int first_mat, int n_mats, double eps, float gram_gain, hipStream_t s) {
  if (n_mats <= 0) return hipSuccess;
  norm_finalize_kernel<<<n_mats, 256, 0, s>>>(mats, first_mat, eps, gram_gain);
  return hipGetLastError();
}

hipError_t launch_apply_update(const MatDesc* mats, const MatPtrs* ptrs, const EwTile* tiles, int n_tiles, float lr, float wd,
                               float rms_scale, int scale_mode, float sqrt_hidden, int o_sel, int use_s, int stream_w,
                               int ns_dtype, hipStream_t s) {
  if (n_tiles <= 0) return hipSuccess;
#define MUON_CALL(XT, PL)                                                                                                          \
  if (stream_w)                                                                                                                    \
    apply_update_kernel<XT, PL, true><<<n_tiles, 256, 0, s>>>(mats, ptrs, tiles, lr, wd, rms_scale, scale_mode, sqrt_hidden, o_sel, \
                                                              use_s);                                                              \
  else                                                                                                                             \
    apply_update_kernel<XT, PL, false><<<n_tiles, 256, 0, s>>>(mats, ptrs, tiles, lr, wd, rms_scale, scale_mode, sqrt_hidden, o_sel, use_s)
  MUON_NS_DISPATCH(ns_dtype, MUON_CALL)
#undef MUON_CALL
  return hipGetLastError();
}

hipError_t launch_update_sumsq(const MatDesc* mats, const EwTile* tiles, int n_tiles, int o_sel, int ns_dtype, hipStream_t s) {
  if (n_tiles <= 0) return hipSuccess;
#define MUON_CALL(XT, PL) update_sumsq_kernel<XT, PL><<<n_tiles, 256, 0, s>>>(mats, tiles, o_sel)
  MUON_NS_DISPATCH(ns_dtype, MUON_CALL)
#undef MUON_CALL
  return hipGetLastError();
}

hipError_t launch_update_rms(const MatDesc* mats, int first_mat, int n_mats, int use_s, int to_scal, float* out, hipStream_t s) {
  if (n_mats <= 0) return hipSuccess;
  update_rms_kernel<<<n_mats, 256, 0, s>>>(mats, first_mat, use_s, to_scal, out);
  return hipGetLastError();
}

hipError_t launch_read_update(const MatDesc* mats, int mat, int o_sel, int use_s, int ns_dtype, void* dst, int dst_dtype,
                              hipStream_t s) {
  const int grid = 1024;
  if (dst_dtype == kDtypeBF16) {
#define MUON_CALL(XT, PL) read_update_kernel<XT, PL, u16><<<grid, 256, 0, s>>>(mats, mat, o_sel, use_s, static_cast<u16*>(dst))
    MUON_NS_DISPATCH(ns_dtype, MUON_CALL)
#undef MUON_CALL
  } else {
#define MUON_CALL(XT, PL) read_update_kernel<XT, PL, float><<<grid, 256, 0, s>>>(mats, mat, o_sel, use_s, static_cast<float*>(dst))
    MUON_NS_DISPATCH(ns_dtype, MUON_CALL)
#undef MUON_CALL
  }
  return hipGetLastError();
}

}  // namespace muon
