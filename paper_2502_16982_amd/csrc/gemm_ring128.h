// 128 x 128 output tile of a Newton-Schulz product for launches that give a compute unit one such tile (device code; the products and
// the operand layouts are described in kernels_gemm_bf16.hip).  Four waves of 64 x 64 on a ring of four 32 KB slabs.
//
// Such a launch is bound by the trip of its slabs from the memory-side cache: with two stages (the tile of the fine launch, which
// shares a compute unit with a second block where there is one) a lone block takes 0.6 us per slab, and 64-wide blocks move twice
// the operands through the LDS.  With four stages three slabs are on their way, 0.29 us per slab at K = 2048 (110 KB/us of operands per
// compute unit; the MFMAs of a slab are 0.22).  The fragments of the next slab are read behind the first half of this slab's MFMAs, the
// requests go out one behind every second MFMA; the addend comes as an image into the first stage that no slab is left for,
// and the results leave from there.  Addresses, swizzles and the order of an element's products are those of the other tiles (same
// bits).  muon_plan.cpp holds the line and both sides' times; us per step: 2560^2 523 -> 440, 1536^2 x 3 369 -> 312, 1408 x 2048 x 3 419 -> 366, 12 of
// 640 x 1408 295 -> 260, 7 of 1024^2 277 -> 250, ragged list of six 296 -> 282.
#pragma once

namespace muon {
namespace {

constexpr int kRing128 = 4;
constexpr size_t kLdsRing128 = (size_t)kRing128 * 2 * 128 * ROWB;

// K >= 256.  ADD: the product has an addend.
template <bool LKM, typename IN, typename OUT, bool ADD>
__device__ __forceinline__ void gemm_ring128_tile(const GemmProblem& p, int row0, int col0, bool diagonal, unsigned char* smem, float beta_acc,
                                                  float beta_e, int alpha_idx, double eps, float diag_add, bool out_f16, float gain) {
  constexpr int BT = 128, NW = 4, F = 2, WT = 64, NST = kRing128;
  constexpr int LREQ = BT / 8 / NW, NLOAD = 2 * LREQ;           // 1 KB requests per wave and slab: L, both
  constexpr int STAGE_B = 2 * BT * ROWB, KSTEPS = BK / 16;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int fr = lane & 31, fh = lane >> 5;

  // ---- requests: a wave instruction fills 8 LDS rows of 128 B, chunks XOR-swizzled by (row / 2) % 8; of the K-major L four k-rows
  // of 256 B, chunks moved by 4 (row % 4)
  constexpr int CPRK = BT / 8, RPK = 64 / CPRK;
  const int dma_row = wave * 8 + (lane >> 3);
  const int dma_chunk = (lane & 7) ^ ((dma_row >> 1) & 7);
  const int km_row = wave * RPK + lane / CPRK;
  const int km_chunk = (lane % CPRK) ^ (4 * (km_row & 3));
  const u16* lsrc = LKM ? static_cast<const u16*>(p.L) + (size_t)km_row * p.ldl + row0 + km_chunk * 8
                        : static_cast<const u16*>(p.L) + (size_t)(row0 + dma_row) * p.ldl + dma_chunk * 8;
  const u16* rsrc = static_cast<const u16*>(p.R) + (size_t)(col0 + dma_row) * p.ldr + dma_chunk * 8;
  const size_t lstep = (size_t)(LKM ? NW * RPK : 8 * NW) * p.ldl, rstep = (size_t)(8 * NW) * p.ldr;
  const size_t lslab = LKM ? (size_t)BK * p.ldl : (size_t)BK;
  const int KT = p.K / BK;
  auto request_one = [&](int kt, int stage, auto n_tag) {
    constexpr int n = decltype(n_tag)::value;
    unsigned char* base = smem + stage * STAGE_B + wave * 1024;
    if constexpr (n < LREQ)
      __builtin_amdgcn_global_load_lds((gptr)(lsrc + n * lstep + (size_t)kt * lslab), (lptr)(base + n * NW * 1024), 16, 0, 0);
    else
      __builtin_amdgcn_global_load_lds((gptr)(rsrc + (n - LREQ) * rstep + (size_t)kt * BK), (lptr)(base + BT * ROWB + (n - LREQ) * NW * 1024), 16, 0, 0);
  };

  // ---- fragment reads (lane addressing as in the other tiles) ----
  const int fkey = (fr >> 1) & 7;
  const unsigned lds0 = (unsigned)(size_t)(lptr)smem;
  const unsigned a_base = (unsigned)((wm * WT + fr) * ROWB), b_base = (unsigned)(BT * ROWB + (wn * WT + fr) * ROWB);
  const int l16 = lane & 15, grp = lane >> 4, r4 = l16 >> 2;
  const unsigned a_km = (unsigned)((8 * (grp >> 1) + r4) * (2 * BT) + (2 * (grp & 1) + ((l16 & 3) >> 1)) * 16 + (l16 & 1) * 8);
  PlaneFrag<F, LKM> fg[2][KSTEPS];               // fragments of two slabs: one multiplied, one being read
  constexpr int RPS = LKM ? 3 * F : 2 * F, NR = KSTEPS * RPS;
  auto read = [&](int stage, auto set_tag, auto n_tag) {
    constexpr int set = decltype(set_tag)::value, kk = decltype(n_tag)::value / RPS, r = decltype(n_tag)::value % RPS;
    PlaneFrag<F, LKM>& f = fg[set][kk];
    const unsigned s = lds0 + (unsigned)(stage * STAGE_B);
    const unsigned chunk = (unsigned)(((2 * kk + fh) ^ fkey) * 16);
    if constexpr (LKM && r < 2 * F)
      lds_read_tr<(16 * kk + 4 * (r & 1)) * 2 * BT>(f.h[r / 2][r & 1], s + a_km + (unsigned)(((wm * (WT / 8) + 4 * (r / 2)) ^ (4 * r4)) * 16));
    else if constexpr (r < RPS - F)
      lds_read<r * 32 * ROWB>(f.a[r], s + a_base + chunk);
    else
      lds_read<(r - RPS + F) * 32 * ROWB>(f.b[r - RPS + F], s + b_base + chunk);
  };
  auto a_frag = [&](const PlaneFrag<F, LKM>& f, int i) -> bf16x8 {
    if constexpr (LKM) {
      const u32x4 both = {f.h[i][0].x, f.h[i][0].y, f.h[i][1].x, f.h[i][1].y};
      return __builtin_bit_cast(bf16x8, both);
    } else {
      return __builtin_bit_cast(bf16x8, f.a[i]);
    }
  };
  f32x16 acc[F][F];
#pragma unroll
  for (int i = 0; i < F; ++i)
#pragma unroll
    for (int j = 0; j < F; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  // The addend's image: 128 rows x 256 B, transposed like the output, chunk of row r at position chunk ^ r % 16.  It comes into the
  // first stage that no slab is left for, and the results leave from the same place.
  constexpr int CPT = BT / 8, RPI = 64 / CPT, NIMG = BT / RPI / NW;
  static_assert(NIMG == NLOAD, "the image is waited for like a slab");
  const u16* Et = static_cast<const u16*>(p.Et);
  auto request_e = [&](int at, auto n_tag) {
    constexpr int n = decltype(n_tag)::value;
    const int r = (n * NW + wave) * RPI + lane / CPT;
    const u16* e = Et + (size_t)(col0 + r) * p.ldet + row0 + ((lane % CPT) ^ (r & 15)) * 8;
    __builtin_amdgcn_global_load_lds((gptr)e, (lptr)(smem + at * STAGE_B + (n * NW + wave) * 1024), 16, 0, 0);
  };

  // One slab (see gemm_tile64_body).  MORE: there is a next slab, with `behind` slabs (the addend's image among them) requested after
  // it.  REFILL: slab kt + NST exists.  SEND_E: the addend's image is requested here.
  int kt = 0, stage = 0;
  auto slab = [&](auto set_tag, auto more_tag, auto refill_tag, auto behind_tag, auto add_tag) {
    constexpr bool SEND_E = decltype(add_tag)::value;
    constexpr int set = decltype(set_tag)::value, behind = decltype(behind_tag)::value;
    constexpr bool MORE = decltype(more_tag)::value, REFILL = decltype(refill_tag)::value;
    asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
#pragma unroll
    for (int kk = 0; kk < KSTEPS; ++kk) tie_planes(fg[set][kk]);
    const int next = stage + 1 == NST ? 0 : stage + 1;
    if constexpr (MORE) {
      wait_vmcnt<NLOAD * behind>();              // my requests of the next slab have landed
      __builtin_amdgcn_s_barrier();              // everybody's; and everybody has read this one
    }
    constexpr int NM = KSTEPS * F * F;
    static_for<0, NM>([&](auto t_tag) {
      constexpr int t = decltype(t_tag)::value, kk = t / (F * F), i = t / F % F, j = t % F;
      if constexpr (MORE) {                      // the reads lead: all of them behind the first half of the MFMAs
        constexpr int half = NM / 2;
        if constexpr (t < half)
          static_for<t * NR / half, (t + 1) * NR / half>([&](auto n_tag) { read(next, std::integral_constant<int, set ^ 1>{}, n_tag); });
      }
      acc[i][j] = IN::mfma(a_frag(fg[set][kk], i), __builtin_bit_cast(bf16x8, fg[set][kk].b[j]), acc[i][j]);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (REFILL)
        static_for<t * NLOAD / NM, (t + 1) * NLOAD / NM>([&](auto n_tag) { request_one(kt + NST, stage, n_tag); });
      if constexpr (SEND_E) static_for<t * NIMG / NM, (t + 1) * NIMG / NM>([&](auto n_tag) { request_e(stage, n_tag); });
      __builtin_amdgcn_sched_barrier(0);
    });
    stage = next;
    ++kt;
  };

  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  using T_ = std::true_type;
  using F_ = std::false_type;
  auto request_slab = [&](int s) { static_for<0, NLOAD>([&](auto n_tag) { request_one(s, s, n_tag); }); };
  auto read_slab = [&](int stage_, auto set_tag) { static_for<0, NR>([&](auto n_tag) { read(stage_, set_tag, n_tag); }); };
  // (extents are padded to 128, so KT is even, and at least four)
  request_slab(0);
  request_slab(1);
  request_slab(2);
  request_slab(3);
  float alpha = 1.f;
  if (!LKM && !ADD && alpha_idx == kAlphaFromPartials) {
    // first Gram product: the norm, from the partial sums (see gemm_tile64_body)
    float s, s2;
    const double sum = block_sum_f64(p.partials, p.n_part, reinterpret_cast<double*>(smem + kLdsRing128));
    norm_scalars(sum, eps, &s, &s2);
    if (row0 == 0 && col0 == 0 && tid == 0) store_norm(const_cast<float*>(p.scal), sum, eps, gain, s, s2);
    alpha = s2;
  } else if (alpha_idx >= 0) {
    alpha = p.scal[alpha_idx];
  }
  wait_vmcnt<NLOAD * (NST - 1)>();
  __builtin_amdgcn_s_barrier();
  read_slab(0, I0{});
  while (kt + NST < KT) {
    slab(I0{}, T_{}, T_{}, I2{}, F_{});
    slab(I1{}, T_{}, T_{}, I2{}, F_{});
  }
  const int image = stage;                       // stage of the addend's and the output's image
  constexpr int e = ADD ? 1 : 0;
  slab(I0{}, T_{}, F_{}, I2{}, std::integral_constant<bool, ADD>{});           // the last four slabs
  slab(I1{}, T_{}, F_{}, std::integral_constant<int, 1 + e>{}, F_{});
  slab(I0{}, T_{}, F_{}, std::integral_constant<int, e>{}, F_{});
  slab(I1{}, F_{}, F_{}, I0{}, F_{});
  wait_vmcnt<0>();
  __syncthreads();                               // every wave has read the last slab, and the addend is there
  unsigned char* const img = smem + image * STAGE_B;

  // ---- epilogue: val = alpha * (beta_acc * acc + beta_e * E) (+ the diagonal constant), in the other tiles' order ----
  const float ab_acc = alpha * beta_acc, ab_e = alpha * beta_e;
  u16* C = static_cast<u16*>(p.C);
  u16* Ct = static_cast<u16*>(p.Ct);
  int ldct = p.ldct;
  if (p.symmetric) {                             // mirror store; the tile itself only off the diagonal
    Ct = C;
    ldct = p.ldc;
    if (diagonal) C = nullptr;
  }
  const int below = (row0 + wm * WT) - (col0 + wn * WT);        // rows minus columns of this wave's MFMA tile (i, j): below + 32 (i - j)
  const bool mirrors = kMayMirror<IN> && !LKM && diagonal && p.symmetric == kMirrored;
  auto slot = [&](int row, int chunk) -> u32x2* {
    return reinterpret_cast<u32x2*>(img + row * (2 * BT) + ((chunk ^ (row & 15)) * 16) + fh * 8);
  };
  u32x2 pk[F][F][4];
  with_output_type<OUT>(out_f16, [&](auto out) {
    using O = decltype(out);
#pragma unroll
    for (int i = 0; i < F; ++i)
#pragma unroll
      for (int j = 0; j < F; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          float x[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) x[e] = ab_acc * acc[i][j][4 * q + e];
          if constexpr (ADD) {
            const u32x2 ev = *slot(wn * WT + 32 * j + fr, (wm * WT + 32 * i) / 8 + q);
            x[0] = fmaf(ab_e, IN::lo(ev.x), x[0]);
            x[1] = fmaf(ab_e, IN::hi(ev.x), x[1]);
            x[2] = fmaf(ab_e, IN::lo(ev.y), x[2]);
            x[3] = fmaf(ab_e, IN::hi(ev.y), x[3]);
          }
          if (p.diag_add != 0 && below + 32 * (i - j) == 0) {
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] += (fr == 8 * q + 4 * fh + e) ? diag_add : 0.f;
          }
          pk[i][j][q] = u32x2{O::pack(x[0], x[1]), O::pack(x[2], x[3])};
        }
  });

  // ---- results leave through the image, 16 bytes per lane ----
  auto store_image = [&](u16* dst, int ld, int first_row, int first_col) {
    u32x4 v[NIMG];
#pragma unroll
    for (int n = 0; n < NIMG; ++n) v[n] = *reinterpret_cast<const u32x4*>(img + (n * NW + wave) * 1024 + lane * 16);
#pragma unroll
    for (int n = 0; n < NIMG; ++n) {
      const int r = (n * NW + wave) * RPI + lane / CPT;
      *(gvec_ptr)(dst + (size_t)(first_row + r) * ld + first_col + ((lane % CPT) ^ (r & 15)) * 8) = v[n];
    }
  };
  const Transposer transposed(fr, fh);
  if (Ct) {
    if (ADD && mirrors) __syncthreads();          // blocks are written that another wave reads the addend from
#pragma unroll
    for (int i = 0; i < F; ++i)
#pragma unroll
      for (int j = 0; j < F; ++j) {
        // kMirrored products on the diagonal: blocks below it are not written, those above it twice
        const int at = below + 32 * (i - j);
        if (mirrors && at > 0) continue;
        if (mirrors && at == 0) mirror_block(transposed, fr, fh, pk[i][j]);
        if (mirrors && at < 0) {
          u32x2 m[4];
          transposed(pk[i][j], m);
#pragma unroll
          for (int q = 0; q < 4; ++q) *slot(wm * WT + 32 * i + fr, (wn * WT + 32 * j) / 8 + q) = m[q];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) *slot(wn * WT + 32 * j + fr, (wm * WT + 32 * i) / 8 + q) = pk[i][j][q];
      }
    __syncthreads();
    store_image(Ct, ldct, col0, row0);
  }
  if (C) {
    if (Ct) __syncthreads();
#pragma unroll
    for (int i = 0; i < F; ++i)
#pragma unroll
      for (int j = 0; j < F; ++j) {
        u32x2 m[4];
        transposed(pk[i][j], m);
#pragma unroll
        for (int q = 0; q < 4; ++q) *slot(wm * WT + 32 * i + fr, (wn * WT + 32 * j) / 8 + q) = m[q];
      }
    __syncthreads();
    store_image(C, p.ldc, row0, col0);
  }
}

// (one branch in front of the tile: a branch while fragment reads are in flight would have their registers copied before they land)
template <bool LKM, typename IN = Bf16, typename OUT = Bf16>
__device__ __forceinline__ void gemm_ring128_body(const GemmProblem& p, int row0, int col0, bool diagonal, unsigned char* smem, float beta_acc,
                                                  float beta_e, int alpha_idx, double eps, float diag_add, bool out_f16 = false,
                                                  float gain = 0.f) {
  if (p.Et) gemm_ring128_tile<LKM, IN, OUT, true>(p, row0, col0, diagonal, smem, beta_acc, beta_e, alpha_idx, eps, diag_add, out_f16, gain);
  else gemm_ring128_tile<LKM, IN, OUT, false>(p, row0, col0, diagonal, smem, beta_acc, beta_e, alpha_idx, eps, diag_add, out_f16, gain);
}

}  // namespace
}  // namespace muon
