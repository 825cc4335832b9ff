// 64 x 64 output tile of a bf16 Newton-Schulz product, for launches that hold few tiles, and 32 x 32 tile of one wave for
// those that hold the fewest (device code; the products and the operand layouts are described in kernels_gemm_bf16.hip, which
// includes this file; split operands: gemm_planes.h).
//
// What bounds such a launch is not the matrix cores but latency: the first operands come from the memory-side cache
// (about 2 us after the block starts), a block's K loop is a serial chain of slabs, and most compute units hold one
// block or none.  So the tile is small - four waves with one 32 x 32 MFMA tile each - and the LDS is a ring of NST
// slabs of 16 KB that are requested as early as a stage is free and waited for with a partial s_waitcnt vmcnt: only the
// first slab's latency is seen.  The fragments of the next slab are read while this one is multiplied; one barrier per slab.
// A ring of three fits a compute unit three times; alone a block waits for its slabs then (0.35 us each: two slabs' time
// is a trip to the memory-side cache), with a ring of four 0.3 us.  One wave by itself (NW = 1) has no barriers, half
// the LDS traffic per slab and a ring of six 8 KB slabs.  muon_plan.cpp holds the line between the three, with their times.
// Addresses, swizzles and the order in which an output element's products are added are those of the large tiles: in
// plain bf16 an element comes out with the same bits whichever tile computes it.
// Measured (us per launch, 256-wide tiles of one block per compute unit / 128-wide tiles / these): Gram product of
// 4 x 1024^2 and 3 x 1024 x 4096 75 / 43 / 34; products of nine matrices of 200 x 333 to 512 x 768 22 / 9 / 6.  Rings of 6 and
// 8 slabs gain no more on lone blocks and cost 5 to 10 % of a step where several blocks could share a compute unit.
#pragma once

namespace muon {
namespace {

constexpr int kRing64 = 3, kRing64Few = 4, kRing32 = 6;
constexpr size_t lds_ring64(int stages) { return (size_t)stages * 128 * ROWB; }
constexpr size_t kLdsRing32 = (size_t)kRing32 * 64 * ROWB;
constexpr size_t kLdsFold64 = 256 * sizeof(double);       // scratch behind the ring for the folded norm

// Fragments of one k-step of a wave, read by assembly (in front of an LDS read of its own the compiler puts a wait for
// all vector memory, the slabs in flight included).  The transposing read of the K-major operand delivers two halves.
template <bool LKM>
struct Frag64 {
  u32x4 a, b;
  u32x2 h0, h1;
};
template <bool LKM, int HALF>     // HALF: bytes from the first half's k-rows to the second's
__device__ __forceinline__ void read64(Frag64<LKM>& f, unsigned a_addr, unsigned b_addr) {
  if constexpr (LKM) {
    asm volatile("ds_read_b64_tr_b16 %0, %1" : "=v"(f.h0) : "v"(a_addr) : "memory");
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(f.h1) : "v"(a_addr), "n"(HALF) : "memory");
  } else {
    asm volatile("ds_read_b128 %0, %1" : "=v"(f.a) : "v"(a_addr) : "memory");
  }
  asm volatile("ds_read_b128 %0, %1" : "=v"(f.b) : "v"(b_addr) : "memory");
}
// The wait for all LDS reads, and a tie of further fragments to the same point of the instruction stream: the covered
// registers are read-write operands, so every MFMA on them depends on the wait.
template <bool LKM>
__device__ __forceinline__ void tie64(Frag64<LKM>& f) {
  if constexpr (LKM) asm volatile("" : "+v"(f.h0), "+v"(f.h1), "+v"(f.b) : : "memory");
  else asm volatile("" : "+v"(f.a), "+v"(f.b) : : "memory");
}
template <bool LKM>
__device__ __forceinline__ void land64(Frag64<LKM>& f) {
  if constexpr (LKM) asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(f.h0), "+v"(f.h1), "+v"(f.b) : : "memory");
  else asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(f.a), "+v"(f.b) : : "memory");
}

// The tile at (row0, col0); `diagonal`: it lies on the diagonal of a symmetric product (its own mirror image).
// IN, OUT, out_f16: as in gemm_tile_body.
template <bool LKM, int NW, int NST, typename IN = Bf16, typename OUT = Bf16>
__device__ __forceinline__ void gemm_tile64_body(const GemmProblem& p, int row0, int col0, bool diagonal, unsigned char* smem,
                                                 float beta_acc, float beta_e, int alpha_idx, double eps, float diag_add,
                                                 bool out_f16 = false, float gain = 0.f) {
  static_assert(NW == 4 || NW == 1, "a wave owns a 32 x 32 tile");
  constexpr int BT = NW == 4 ? 64 : 32;                         // tile side
  constexpr int LREQ = BT / 8 / NW, NLOAD = 2 * LREQ;           // 1 KB requests per wave and slab: L, both
  constexpr int STAGE_B = 2 * BT * ROWB, KSTEPS = BK / 16;
  static_assert(NST >= 2 && NLOAD * (NST - 1) < 64, "ring shape");
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = NW == 4 ? wave >> 1 : 0, wn = NW == 4 ? wave & 1 : 0;
  const int fr = lane & 31, fh = lane >> 5;

  // ---- requests: a wave instruction fills 8 LDS rows of 128 B (L rows or R rows), which keep their 16-byte chunks
  // XOR-swizzled by (row / 2) % 8; or, of the K-major L, 1 KB of 64 k-rows of 2 BT bytes, whose chunks are moved by
  // 4 ((row / 2) % 2) where rows are 128 B (it spreads the four k-rows one transposing read touches over the banks; four rows
  // of 64 B do not meet).
  constexpr int CPRK = BT / 8, RPK = 64 / CPRK;
  const int dma_row = wave * 8 + (lane >> 3);
  const int dma_chunk = (lane & 7) ^ ((dma_row >> 1) & 7);      // of request 0; one wave: odd requests start 8 rows on, key + 4
  const int km_row = wave * RPK + lane / CPRK;
  const int km_chunk = (lane % CPRK) ^ (NW == 4 ? 4 * ((km_row >> 1) & 1) : 0);
  const u16* lsrc = LKM ? static_cast<const u16*>(p.L) + (size_t)km_row * p.ldl + row0 + km_chunk * 8
                        : static_cast<const u16*>(p.L) + (size_t)(row0 + dma_row) * p.ldl + dma_chunk * 8;
  const u16* rsrc = static_cast<const u16*>(p.R) + (size_t)(col0 + dma_row) * p.ldr + dma_chunk * 8;
  const int odd = NW == 4 ? 0 : (dma_chunk ^ 4) * 8 - dma_chunk * 8;
  const size_t lstep = (size_t)(LKM ? NW * RPK : 8 * NW) * p.ldl, rstep = (size_t)(8 * NW) * p.ldr;
  const size_t lslab = LKM ? (size_t)BK * p.ldl : (size_t)BK;
  const int KT = p.K / BK;
  auto request_one = [&](int kt, int stage, auto n_tag) {
    constexpr int n = decltype(n_tag)::value;
    unsigned char* base = smem + stage * STAGE_B + wave * 1024;
    if constexpr (n < LREQ)
      __builtin_amdgcn_global_load_lds((gptr)(lsrc + n * lstep + (size_t)kt * lslab + (!LKM && n % 2 ? odd : 0)), (lptr)(base + n * NW * 1024), 16, 0, 0);
    else
      __builtin_amdgcn_global_load_lds((gptr)(rsrc + (n - LREQ) * rstep + (size_t)kt * BK + ((n - LREQ) % 2 ? odd : 0)),
                                       (lptr)(base + BT * ROWB + (n - LREQ) * NW * 1024), 16, 0, 0);
  };

  // ---- fragment reads (lane addressing as in the large tiles) ----
  const int fkey = (fr >> 1) & 7;
  const unsigned lds0 = (unsigned)(size_t)(lptr)smem;
  const unsigned a_base = (unsigned)((wm * 32 + fr) * ROWB), b_base = (unsigned)(BT * ROWB + (wn * 32 + fr) * ROWB);
  const int l16 = lane & 15, grp = lane >> 4, r4 = l16 >> 2;
  const unsigned a_km = (unsigned)((8 * (grp >> 1) + r4) * (2 * BT) +
                                   (((4 * wm) ^ (NW == 4 ? 4 * ((r4 >> 1) & 1) : 0)) + 2 * (grp & 1) + ((l16 & 3) >> 1)) * 16 + (l16 & 1) * 8);
  Frag64<LKM> fg[2][KSTEPS];                     // fragments of two slabs: one multiplied, one being read
  auto read_slab = [&](int stage, auto set_tag) {
    constexpr int set = decltype(set_tag)::value;
    const unsigned sa = lds0 + (unsigned)(stage * STAGE_B);
    static_for<0, KSTEPS>([&](auto kk_tag) {
      constexpr int kk = decltype(kk_tag)::value;
      const unsigned chunk = (unsigned)(((2 * kk + fh) ^ fkey) * 16);
      read64<LKM, 4 * 2 * BT>(fg[set][kk], LKM ? sa + (unsigned)(16 * kk * 2 * BT) + a_km : sa + a_base + chunk, sa + b_base + chunk);
    });
  };
  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;

  // One slab, whose fragments are in set `set` or on their way there.  MORE: there is a next slab, with `behind` slabs
  // requested after it; its fragments are read into the other set while this slab is multiplied.  REFILL: slab kt + NST
  // exists and goes into this slab's stage, which every wave has read when the barrier opens; a request holds the
  // wave's in-order issue port until the memory pipeline takes it, so each goes out behind an MFMA.
  int kt = 0, stage = 0;
  auto slab = [&](auto set_tag, auto more_tag, auto refill_tag, auto behind_tag) {
    constexpr int set = decltype(set_tag)::value, behind = decltype(behind_tag)::value;
    constexpr bool MORE = decltype(more_tag)::value, REFILL = decltype(refill_tag)::value;
    land64(fg[set][0]);
#pragma unroll
    for (int kk = 1; kk < KSTEPS; ++kk) tie64(fg[set][kk]);
    const int next = stage + 1 == NST ? 0 : stage + 1;
    if constexpr (MORE) {
      wait_vmcnt<NLOAD * behind>();              // my requests of the next slab have landed
      __builtin_amdgcn_s_barrier();              // everybody's; and everybody has read this one
      read_slab(next, std::integral_constant<int, set ^ 1>{});
    }
    static_for<0, KSTEPS>([&](auto kk_tag) {
      constexpr int kk = decltype(kk_tag)::value;
      bf16x8 a;
      if constexpr (LKM) {
        const u32x4 both = {fg[set][kk].h0.x, fg[set][kk].h0.y, fg[set][kk].h1.x, fg[set][kk].h1.y};
        a = __builtin_bit_cast(bf16x8, both);
      } else {
        a = __builtin_bit_cast(bf16x8, fg[set][kk].a);
      }
      acc = IN::mfma(a, __builtin_bit_cast(bf16x8, fg[set][kk].b), acc);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (REFILL)
        static_for<kk * NLOAD / KSTEPS, (kk + 1) * NLOAD / KSTEPS>([&](auto n_tag) { request_one(kt + NST, stage, n_tag); });
    });
    stage = next;
    ++kt;
  };

  // ---- the addend: this lane's pieces of its MFMA tile, 8 contiguous bytes each of the transposed addend, requested ahead of
  // the first slab; being older than every slab they are never counted in a wait for one.
  const u16* Et = static_cast<const u16*>(p.Et);
  const bool has_e = Et != nullptr;
  u32x2 ev[4];
  if (has_e) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      ev[q] = *reinterpret_cast<const u32x2*>(Et + (size_t)(col0 + wn * 32 + fr) * p.ldet + row0 + wm * 32 + 8 * q + 4 * fh);
  }

  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using T_ = std::true_type;
  using F_ = std::false_type;
  auto request_slab = [&](int s) { static_for<0, NLOAD>([&](auto n_tag) { request_one(s, s, n_tag); }); };
  // (extents are padded to 128, so KT is even)
  request_slab(0);
  request_slab(1);
  if constexpr (NST % 2 == 0)
    static_for<2, NST>([&](auto s_tag) {
      if (decltype(s_tag)::value < KT) request_slab(decltype(s_tag)::value);
    });
  float alpha = 1.f;
  if (!LKM && alpha_idx == kAlphaFromPartials) {
    // first Gram product: the norm, from the partial sums (K-major launches are never first)
    float s, s2;
    double sum;
    if constexpr (NW == 4) sum = block_sum_f64(p.partials, p.n_part, reinterpret_cast<double*>(smem + lds_ring64(NST)));
    else sum = wave_sum_f64(p.partials, p.n_part);
    norm_scalars(sum, eps, &s, &s2);
    if (row0 == 0 && col0 == 0 && tid == 0) store_norm(const_cast<float*>(p.scal), sum, eps, gain, s, s2);
    alpha = s2;
  } else if (alpha_idx >= 0) {
    alpha = p.scal[alpha_idx];
  }
  if constexpr (NST == 3) {
    if (KT == 2) {                               // K = 128: all of it is on its way
      wait_vmcnt<NLOAD>();
      __builtin_amdgcn_s_barrier();
      read_slab(0, I0{});
      slab(I0{}, T_{}, F_{}, I0{});
      slab(I1{}, F_{}, F_{}, I0{});
    } else {
      request_slab(2);
      wait_vmcnt<2 * NLOAD>();
      __builtin_amdgcn_s_barrier();
      read_slab(0, I1{});
      slab(I1{}, T_{}, T_{}, I1{});
      while (kt + NST < KT) {
        slab(I0{}, T_{}, T_{}, I1{});
        slab(I1{}, T_{}, T_{}, I1{});
      }
      slab(I0{}, T_{}, F_{}, I1{});
      slab(I1{}, T_{}, F_{}, I0{});
      slab(I0{}, F_{}, F_{}, I0{});
    }
  } else {
    static_assert(NST == 4 || NST == 6, "every shorter K has its wait");
    if (KT >= NST) wait_vmcnt<NLOAD * (NST - 1)>();
    else if (KT == 4) wait_vmcnt<NLOAD * 3>();
    else wait_vmcnt<NLOAD>();
    __builtin_amdgcn_s_barrier();
    read_slab(0, I0{});
    while (kt + NST < KT) {
      slab(I0{}, T_{}, T_{}, std::integral_constant<int, NST - 2>{});
      slab(I1{}, T_{}, T_{}, std::integral_constant<int, NST - 2>{});
    }
    static_for<0, NST / 2>([&](auto h_tag) {
      constexpr int left = NST - 1 - 2 * decltype(h_tag)::value;               // slabs behind this one
      if (left == 1 || KT > left) {
        slab(I0{}, T_{}, F_{}, std::integral_constant<int, left - 1>{});
        slab(I1{}, std::integral_constant<bool, (left > 1)>{}, F_{}, std::integral_constant<int, (left > 1 ? left - 2 : 0)>{});
      }
    });
  }
  __syncthreads();                               // every wave has read the last slab: the LDS is free for the images

  // ---- epilogue: val = alpha * (beta_acc * acc + beta_e * E) (+ the diagonal constant), in the large tiles' order ----
  const float ab_acc = alpha * beta_acc, ab_e = alpha * beta_e;
  u16* C = static_cast<u16*>(p.C);
  u16* Ct = static_cast<u16*>(p.Ct);
  int ldct = p.ldct;
  if (p.symmetric) {                             // mirror store; the tile itself only off the diagonal
    Ct = C;
    ldct = p.ldc;
    if (diagonal) C = nullptr;
  }
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] *= ab_acc;
  if (has_e) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      acc[4 * q + 0] = fmaf(ab_e, IN::lo(ev[q].x), acc[4 * q + 0]);
      acc[4 * q + 1] = fmaf(ab_e, IN::hi(ev[q].x), acc[4 * q + 1]);
      acc[4 * q + 2] = fmaf(ab_e, IN::lo(ev[q].y), acc[4 * q + 2]);
      acc[4 * q + 3] = fmaf(ab_e, IN::hi(ev[q].y), acc[4 * q + 3]);
    }
  }
  if (p.diag_add != 0 && row0 + wm * 32 == col0 + wn * 32) {     // wave-uniform
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] += (fr == 8 * (v >> 2) + 4 * fh + (v & 3)) ? diag_add : 0.f;
  }

  // ---- results leave through swizzled LDS images of 64 rows x 128 B (chunk of row r at position
  // chunk ^ (r / 2) % 8), 16 bytes per lane ----
  constexpr int CPT = BT / 8, RPI = 64 / CPT, NIMG = BT / RPI / NW;     // chunks per row, rows and instructions per wave
  auto key = [](int row) { return NW == 4 ? (row >> 1) & 7 : (row >> 2) & 3; };
  auto slot = [&](int row, int chunk) -> u32x2* {
    return reinterpret_cast<u32x2*>(smem + row * (2 * BT) + ((chunk ^ key(row)) * 16) + fh * 8);
  };
  auto store_image = [&](u16* dst, int ld, int first_row, int first_col) {
    u32x4 v[NIMG];
#pragma unroll
    for (int n = 0; n < NIMG; ++n) v[n] = *reinterpret_cast<const u32x4*>(smem + (n * NW + wave) * 1024 + lane * 16);
#pragma unroll
    for (int n = 0; n < NIMG; ++n) {
      const int r = (n * NW + wave) * RPI + lane / CPT;
      *(gvec_ptr)(dst + (size_t)(first_row + r) * ld + first_col + ((lane % CPT) ^ key(r)) * 8) = v[n];
    }
  };
  bf16x8 sel[2];                                 // 0/1 selector of the MFMA transpose
#pragma unroll
  for (int sx = 0; sx < 2; ++sx)
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int row = 16 * sx + 4 * fh + (t < 4 ? t : 4 + t);
      sel[sx][t] = (__bf16)(fr == row ? 1.0f : 0.0f);
    }
  auto pack2f = [](float x, float y) {
    const f32x2 v = {x, y};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
  };
  u32x2 pk[4];
  with_output_type<OUT>(out_f16, [&](auto out) {
    using O = decltype(out);
#pragma unroll
    for (int q = 0; q < 4; ++q) pk[q] = u32x2{O::pack(acc[4 * q], acc[4 * q + 1]), O::pack(acc[4 * q + 2], acc[4 * q + 3])};
  });
  // kMirrored product, tile on the diagonal: the wave below it writes nothing, the one above it both blocks
  const bool mirrors = kMayMirror<IN> && !LKM && diagonal && p.symmetric == kMirrored;
  if constexpr (kMayMirror<IN> && !LKM) {
    if (mirrors && wm <= wn) {
      const Transposer transposed(fr, fh);
      if (wm == wn) {
        mirror_block(transposed, fr, fh, pk);
      } else {
        u32x2 m[4];
        transposed(pk, m);
#pragma unroll
        for (int q = 0; q < 4; ++q) *slot(wm * 32 + fr, 4 * wn + q) = m[q];
      }
    }
  }
  if (Ct) {
    if (!mirrors || wm <= wn) {
#pragma unroll
      for (int q = 0; q < 4; ++q) *slot(wn * 32 + fr, 4 * wm + q) = pk[q];
    }
    __syncthreads();
    store_image(Ct, ldct, col0, row0);
  }
  if (C) {
    if (Ct) __syncthreads();
    f32x16 d;
#pragma unroll
    for (int v = 0; v < 16; ++v) d[v] = 0.f;
#pragma unroll
    for (int sx = 0; sx < 2; ++sx) {
      const u32x4 raw = {pk[2 * sx].x, pk[2 * sx].y, pk[2 * sx + 1].x, pk[2 * sx + 1].y};
      d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, raw), sel[sx], d, 0, 0, 0);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
      *slot(wm * 32 + fr, 4 * wn + q) = u32x2{pack2f(d[4 * q], d[4 * q + 1]), pack2f(d[4 * q + 2], d[4 * q + 3])};
    __syncthreads();
    store_image(C, p.ldc, row0, col0);
  }
}

}  // namespace
}  // namespace muon
