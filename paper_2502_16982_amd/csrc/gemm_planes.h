// Output tile of a Newton-Schulz product of split operands: every matrix is the sum of PL = 2 or 3 bf16 planes (device code;
// the products, the operand layouts and the meaning of the planes are described in kernels_gemm_bf16.hip, which includes this
// file).  BT = 64 or 128: side of the tile, four waves of (BT / 2)^2.
//
// The plane pairs (i, j) with i + j < PL of one 64-wide piece of K are multiplied while the piece is at hand.  A "unit" is
// one plane of one piece, L and R rows together; units come plane 0, 1, .. of a piece, then the next piece.  A wave keeps the
// fragments of the planes it has read until the piece is done, and unit q adds the pairs whose larger plane is q: (0,0); then
// (1,0), (0,1) and with three planes (1,1); then (2,0), (0,2).  So every plane passes through the memory path and the LDS
// once per piece: 4 operand panels against 6 in a loop over the pairs (PL = 2), 6 against 12 (PL = 3), and a 64-wide wave tile
// reads 85 and 64 B of LDS per clock of MFMAs instead of 128.  What bounds the launches now, in shares of the cycles in which a
// compute unit has work, matrix cores / LDS reads: width-1024 layer with two planes, Gram product in 64-wide tiles 0.51 / 0.36, apply
// product in 128-wide ones 0.63 / 0.27; coarse tables of the 4096-wide block 0.74 to 0.75 / 0.27, which is power.
// The LDS is a ring of NST units, requested as early as a stage is free and waited for with a partial s_waitcnt vmcnt; the
// next unit's fragments are read while this one is multiplied; one barrier per unit.  The addend's planes come through the
// same ring behind the last unit.  BT = 64: three stages, or four where a launch leaves a block alone on its compute unit: one
// more unit in flight (two planes: 512^2 118 -> 109 us, 1024 x 4096 397 -> 362, 5 of 40 x 3800 222 -> 189; three: 156 -> 145, 579
// -> 545, 307 -> 265), but fewer blocks on a compute unit (10 of 512^2 208 -> 214 and 292 -> 296).  BT = 128: three planes
// take the registers of a whole compute unit, ring of 4.  Two planes fit two blocks with a ring of 2 (250 registers), or one with a
// ring of 4 and three accumulators: the symmetric products of large matrices, the coarse tables, run like that, us per launch two
// blocks / one: Gram 8192^2 1530 / 1450, 2 of 4096 x 11008 1039 / 967, 4 of 2048 x 8192 489 / 429, 3 of 3200^2 272 / 278;
// everything else runs two (apply product of 12 of 1536 x 8192 1231 / 1399, steps of lists of 512^2 to 1024 x 4096 +8 to +20 %).
// Rounding.  Three planes, and two with the ring of 4: the leading pair has two accumulators, of even and odd pieces, and the
// other pairs a third, so the small terms are not rounded at the size of the sum (error of O against 64 bits, three planes:
// 1024 x 4096 1.38e-6 -> 0.97e-6, 100 x 300 6.4e-7 -> 5.9e-7 against one accumulator that takes the pairs one after the other,
// smallest first).  Two planes with one accumulator: +0.3 to +1 % of the error.
// Two planes: the polynomial takes the pair (1,1) too, whose 2^-18 is as large as the rounding of the second plane (512^2
// 2.20e-5 -> 2.13e-5, 1024 x 4096 2.14e-5 -> 1.87e-5).  All of that comes from the diagonal of A, the part of A A^T's sums that does
// not average: the coarse tables, where a quarter of the products shows, take the pair only in the pieces of K that hold the tile's
// own rows or columns.  Error of O before the pair / with it / in own pieces and three accumulators: 4096^2 1.72e-5 / 1.68e-5 /
// 1.67e-5, 4096 x 11008 2.33e-5 / 1.48e-5 / 1.42e-5, 8192^2 1.67e-5 / 1.63e-5 / 1.60e-5; us per polynomial launch: 8 of 4096^2 1659 /
// 1899 / 1568, 8192^2 1480 / 1898 / 1458.  (On shorter lists own pieces are 2 to 5 % of a step faster and the error 0.1 to 0.4 %
// larger: they take the whole pair.)
// Measured, us per step, with 256- and 128-wide tiles in a loop over pairs / now.  Two planes: 4 of 1024^2 with 3 of 1024 x 4096
// 1306 / 1066, 48 of 1024^2 4173 / 3717, 12 of 1536 x 8192 12599 / 10800, 3 of 16 x 2000 206 / 145, 7 of 4096^2 27013 / 25770, 4
// of 4096^2 with 3 of 4096 x 11008 41783 / 39316, 8192^2 28525 / 28525.  Three planes: 4096^2 8970 / 7052, 24 of 1024 x 4096
// 12377 / 9707, 30 of 300 x 700 840 / 660, ten iterations of 4 of 512^2, 2 of 512 x 1536 and 1500 x 500 1210 / 673.
#pragma once

namespace muon {
namespace {

constexpr int planes_ring(int bt, int pl) { return bt == 64 ? 3 : pl == 2 ? 2 : 4; }
constexpr int kPlanesRingFew = 4;                // BT = 64 where a block has a compute unit to itself
constexpr int planes_ring_coarse(bool kmajor, int pl) { return pl == 2 && !kmajor ? 4 : planes_ring(128, pl); }
constexpr size_t planes_lds(int bt, int stages) { return (size_t)stages * 2 * (size_t)bt * ROWB; }

// Fragments of one k-step of one plane, read by assembly (see gemm_tile64.h).
template <int F, bool LKM>
struct PlaneFrag {
  u32x4 a[F], b[F];
  u32x2 h[F][2];
};
template <int OFFSET>
__device__ __forceinline__ void lds_read(u32x4& v, unsigned addr) {
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFFSET) : "memory");
}
template <int OFFSET>
__device__ __forceinline__ void lds_read_tr(u32x2& v, unsigned addr) {
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFFSET) : "memory");
}
template <int F, bool LKM>
__device__ __forceinline__ void tie_planes(PlaneFrag<F, LKM>& f) {
#pragma unroll
  for (int i = 0; i < F; ++i) {
    if constexpr (LKM) asm volatile("" : "+v"(f.h[i][0]), "+v"(f.h[i][1]), "+v"(f.b[i]) : : "memory");
    else asm volatile("" : "+v"(f.a[i]), "+v"(f.b[i]) : : "memory");
  }
}

// ADD: the product has an addend.  The tile at (row0, col0); `diagonal`: it lies on the diagonal of a symmetric product (its own mirror image).
template <int BT, int NST, bool LKM, int PL, bool ADD>
__device__ __forceinline__ void gemm_planes_body(const GemmProblem& p, int row0, int col0, bool diagonal, unsigned char* smem,
                                                 float beta_acc, float beta_e, int alpha_idx, double eps) {
  constexpr int NW = 4, F = BT / 64, WT = BT / 2;
  constexpr int LREQ = BT / 32, NLOAD = 2 * LREQ;               // 1 KB requests per wave and unit: L, both
  constexpr bool SPLIT = PL == 3 || (BT == 128 && NST == 4);    // three accumulators
  constexpr bool OWN11 = PL == 2 && SPLIT && !LKM && ADD, ALL11 = !OWN11 && (PL == 3 || (!LKM && ADD));
  constexpr int UNIT_B = 2 * BT * ROWB, KSTEPS = BK / 16, NACC = SPLIT ? 3 : 1;
  static_assert((BT == 64 || BT == 128) && NST >= PL && NST <= 2 * PL && NLOAD * (NST - 1) < 64, "ring shape");
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int fr = lane & 31, fh = lane >> 5;

  // ---- requests: a wave instruction fills 8 LDS rows of 128 B, chunks XOR-swizzled by (row / 2) % 8; of the K-major L 64
  // k-rows of 2 BT bytes, whose chunks are moved by 4 ((row / 2) % 2) (BT = 64) or 4 (row % 4), which spreads the four k-rows
  // one transposing read touches over the banks.
  constexpr int CPRK = BT / 8, RPK = 64 / CPRK;
  const int dma_row = wave * 8 + (lane >> 3);
  const int dma_chunk = (lane & 7) ^ ((dma_row >> 1) & 7);
  const int km_row = wave * RPK + lane / CPRK;
  const int km_chunk = (lane % CPRK) ^ (4 * (BT == 64 ? (km_row >> 1) & 1 : km_row & 3));
  const u16* lsrc = LKM ? static_cast<const u16*>(p.L) + (size_t)km_row * p.ldl + row0 + km_chunk * 8
                        : static_cast<const u16*>(p.L) + (size_t)(row0 + dma_row) * p.ldl + dma_chunk * 8;
  const u16* rsrc = static_cast<const u16*>(p.R) + (size_t)(col0 + dma_row) * p.ldr + dma_chunk * 8;
  const size_t lstep = (size_t)(LKM ? NW * RPK : 8 * NW) * p.ldl, rstep = (size_t)(8 * NW) * p.ldr;
  const size_t lpiece = LKM ? (size_t)BK * p.ldl : (size_t)BK;
  const int pieces = p.K / BK;                   // extents are padded to 128: at least 2
  // requests [first, first + count) of plane q of a piece
  auto request = [&](int piece, auto q_tag, int stage, auto first_tag, auto count_tag) {
    constexpr int q = decltype(q_tag)::value, first = decltype(first_tag)::value, count = decltype(count_tag)::value;
    unsigned char* base = smem + stage * UNIT_B + wave * 1024;
    const u16* l = lsrc + (size_t)piece * lpiece + (size_t)q * (size_t)p.l_plane;
    const u16* r = rsrc + (size_t)piece * BK + (size_t)q * (size_t)p.r_plane;
    static_for<first, first + count>([&](auto n_tag) {
      constexpr int n = decltype(n_tag)::value;
      if constexpr (n < LREQ)
        __builtin_amdgcn_global_load_lds((gptr)(l + n * lstep), (lptr)(base + n * NW * 1024), 16, 0, 0);
      else
        __builtin_amdgcn_global_load_lds((gptr)(r + (n - LREQ) * rstep), (lptr)(base + BT * ROWB + (n - LREQ) * NW * 1024), 16, 0, 0);
    });
  };

  // ---- fragment reads (lane addressing as in the other tiles) ----
  const int fkey = (fr >> 1) & 7;
  const unsigned lds0 = (unsigned)(size_t)(lptr)smem;
  const unsigned a_base = (unsigned)((wm * WT + fr) * ROWB), b_base = (unsigned)(BT * ROWB + (wn * WT + fr) * ROWB);
  const int l16 = lane & 15, grp = lane >> 4, r4 = l16 >> 2;
  const int km_key = 4 * (BT == 64 ? (r4 >> 1) & 1 : r4);
  const unsigned a_km = (unsigned)((8 * (grp >> 1) + r4) * (2 * BT) + (2 * (grp & 1) + ((l16 & 3) >> 1)) * 16 + (l16 & 1) * 8);
  PlaneFrag<F, LKM> fg[PL][KSTEPS];
  constexpr int RPS = LKM ? 3 * F : 2 * F;       // reads per k-step: the L side's first
  auto read = [&](int stage, auto q_tag, auto n_tag) {          // read n of unit q: k-step n / RPS
    constexpr int q = decltype(q_tag)::value, kk = decltype(n_tag)::value / RPS, r = decltype(n_tag)::value % RPS;
    PlaneFrag<F, LKM>& f = fg[q][kk];
    const unsigned s = lds0 + (unsigned)(stage * UNIT_B);
    const unsigned chunk = (unsigned)(((2 * kk + fh) ^ fkey) * 16);
    if constexpr (LKM && r < 2 * F)
      lds_read_tr<(16 * kk + 4 * (r & 1)) * 2 * BT>(f.h[r / 2][r & 1], s + a_km + (unsigned)(((wm * (WT / 8) + 4 * (r / 2)) ^ km_key) * 16));
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
  f32x16 acc[NACC][F][F];
#pragma unroll
  for (int c = 0; c < NACC; ++c)
#pragma unroll
    for (int i = 0; i < F; ++i)
#pragma unroll
      for (int j = 0; j < F; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[c][i][j][v] = 0.f;

  // Output images, BT rows x 2 BT bytes, one per plane at the start of a ring stage; 16-byte chunks of a row XOR-swizzled by
  // key(row).  A lane owns 8-byte pieces of an image, the same ones of every image.  The addend's planes, transposed like
  // the output, are requested as PL further units into the images' places, and replaced there by the results.
  constexpr int CPT = BT / 8, RPI = 64 / CPT, NIMG = BT / RPI / NW;     // chunks per row, rows and instructions per wave
  static_assert(UNIT_B >= BT * 2 * BT, "an image fits a stage");
  auto key = [](int row) { return BT == 64 ? (row >> 1) & 7 : row & 15; };
  const u16* Et = static_cast<const u16*>(p.Et);
  auto request_e = [&](auto q_tag, int at, auto first_tag, auto count_tag) {
    constexpr int q = decltype(q_tag)::value, first = decltype(first_tag)::value, count = decltype(count_tag)::value;
    const int l = thread_index(0);               // worked out anew: it would take registers from the main loop
    static_for<first, first + count>([&](auto n_tag) {
      constexpr int n = decltype(n_tag)::value;
      const int r = (n * NW + wave) * RPI + l / CPT;
      const u16* e = Et + (size_t)q * (size_t)p.et_plane + (size_t)(col0 + r) * p.ldet + row0 + ((l % CPT) ^ key(r)) * 8;
      __builtin_amdgcn_global_load_lds((gptr)e, (lptr)(smem + at * UNIT_B + (n * NW + wave) * 1024), 16, 0, 0);
    });
  };

  // Pieces of K that hold rows of this tile's own row or column range (the polynomial, whose K runs over the rows of A).
  auto own = [&](int piece) { return (unsigned)(piece * BK - row0) < (unsigned)BT || (unsigned)(piece * BK - col0) < (unsigned)BT; };
  // Unit (piece, q), whose fragments are on their way; LEFT units follow it (kMany: enough for everything).  Its first k-step
  // is multiplied as soon as its fragments have landed; then one wait and barrier: all of this unit's fragments are in
  // registers, everybody's, and the next unit is in the LDS.  From there on, spread among the MFMAs, the next unit's fragments
  // are read - those of plane 0, whose predecessors this unit still needs, a k-step behind - and the unit NST further on is
  // requested into this unit's stage: a request holds the wave's in-order issue port until the memory pipeline takes it.  The
  // addend's planes follow the last unit.
  constexpr int kMany = 1 << 20;
  int stage = 0;
  auto unit = [&](int piece, auto odd_tag, auto q_tag, auto left_tag) {
    constexpr int q = decltype(q_tag)::value, left = decltype(left_tag)::value, next_q = (q + 1) % PL;
    constexpr int e = NST - 1 - left;            // plane of the addend that goes out here
    constexpr bool REFILL = left >= NST, REFILL_E = ADD && !REFILL && e < PL;
    // requests that may be outstanding behind the next unit's: units after it, planes of the addend after those
    constexpr int units_behind = left == 0 ? 0 : left - 1 < NST - 2 ? left - 1 : NST - 2;
    constexpr int adds_behind = ADD && left > 0 ? (NST - 2 - units_behind < PL ? NST - 2 - units_behind : PL) : 0;
    // pairs whose larger plane is q, and MFMA t of a k-step: pair t / F^2, tile (t / F % F, t % F)
    constexpr int pairs = q == 0 ? 1 : q == 1 && ALL11 ? 3 : 2, NM = pairs * F * F;
    auto mma = [&](auto kk_tag, auto t_tag) {
      constexpr int kk = decltype(kk_tag)::value, t = decltype(t_tag)::value, pair = t / (F * F), i = t / F % F, j = t % F;
      constexpr int lp = pair == 0 || pair == 2 ? q : 0, rp = pair == 0 ? 0 : q;
      constexpr int c = !SPLIT ? 0 : q > 0 ? 2 : decltype(odd_tag)::value;
      acc[c][i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a_frag(fg[lp][kk], i), __builtin_bit_cast(bf16x8, fg[rp][kk].b[j]),
                                                             acc[c][i][j], 0, 0, 0);
    };
    asm volatile("s_waitcnt lgkmcnt(%0)" : : "n"((KSTEPS - 1) * RPS < 15 ? (KSTEPS - 1) * RPS : 15) : "memory");
    tie_planes(fg[q][0]);
    __builtin_amdgcn_sched_barrier(0);
    static_for<0, NM>([&](auto t_tag) { mma(std::integral_constant<int, 0>{}, t_tag); });
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
#pragma unroll
    for (int kk = 1; kk < KSTEPS; ++kk) tie_planes(fg[q][kk]);
    const int next = stage + 1 == NST ? 0 : stage + 1;
    if constexpr (left > 0) wait_vmcnt<NLOAD * units_behind + NIMG * adds_behind>();   // my requests of the next unit have landed
    if constexpr (left > 0 || REFILL_E) __builtin_amdgcn_s_barrier();                   // everybody's; and everybody has read this one
    constexpr int ALL = (KSTEPS - 1) * NM, NR = KSTEPS * RPS;
    static_for<0, ALL>([&](auto at_tag) {
      constexpr int at = decltype(at_tag)::value;
      mma(std::integral_constant<int, 1 + at / NM>{}, std::integral_constant<int, at % NM>{});
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (left > 0) {
        // plane 0: k-steps 0 .. KSTEPS-2 here, in step with the MFMAs of 1 .. KSTEPS-1
        constexpr int total = next_q == 0 ? NR - RPS : NR;
        static_for<at * total / ALL, (at + 1) * total / ALL>([&](auto n_tag) { read(next, std::integral_constant<int, next_q>{}, n_tag); });
      }
      if constexpr (REFILL)
        request(piece + (q + NST) / PL, std::integral_constant<int, (q + NST) % PL>{}, stage, std::integral_constant<int, at * NLOAD / ALL>{},
                std::integral_constant<int, (at + 1) * NLOAD / ALL - at * NLOAD / ALL>{});
      if constexpr (REFILL_E)
        request_e(std::integral_constant<int, REFILL_E ? e : 0>{}, stage, std::integral_constant<int, at * NIMG / ALL>{},
                  std::integral_constant<int, (at + 1) * NIMG / ALL - at * NIMG / ALL>{});
      __builtin_amdgcn_sched_barrier(0);
    });
    if constexpr (left > 0 && next_q == 0)
      static_for<NR - RPS, NR>([&](auto n_tag) { read(next, std::integral_constant<int, 0>{}, n_tag); });
    if constexpr (OWN11 && q == 1)
      if (own(piece)) {                          // the pair (1,1): its fragments stay until the next unit of this plane
        static_for<0, KSTEPS * F * F>([&](auto t_tag) {
          constexpr int t = decltype(t_tag)::value, kk = t / (F * F), i = t / F % F, j = t % F;
          acc[NACC - 1][i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a_frag(fg[q][kk], i), __builtin_bit_cast(bf16x8, fg[q][kk].b[j]),
                                                                        acc[NACC - 1][i][j], 0, 0, 0);
        });
        __builtin_amdgcn_sched_barrier(0);
      }
    stage = next;
  };

  static_for<0, NST>([&](auto u_tag) {
    constexpr int u = decltype(u_tag)::value;
    request(u / PL, std::integral_constant<int, u % PL>{}, u, std::integral_constant<int, 0>{}, std::integral_constant<int, NLOAD>{});
  });
  float alpha = 1.f;
  if (BT == 64 && !LKM && alpha_idx == kAlphaFromPartials) {
    // first Gram product: the norm, from the partial sums (K-major launches are never first)
    float s, s2;
    norm_scalars(block_sum_f64(p.partials, p.n_part, reinterpret_cast<double*>(smem + planes_lds(BT, NST))), eps, &s, &s2);
    if (row0 == 0 && col0 == 0 && tid == 0) {
      float* scal = const_cast<float*>(p.scal);
      scal[0] = s;
      scal[1] = s2;
    }
    alpha = s2;
  } else if (alpha_idx >= 0) {
    alpha = p.scal[alpha_idx];
  }
  wait_vmcnt<NLOAD * (NST - 1)>();
  __builtin_amdgcn_s_barrier();
  static_for<0, KSTEPS * RPS>([&](auto n_tag) { read(0, std::integral_constant<int, 0>{}, n_tag); });
  int piece = 0;
  constexpr int STEP = SPLIT ? 2 : 1;            // pieces per pass of the loop (their number is even)
  for (; piece + 2 < pieces; piece += STEP)
    static_for<0, STEP * PL>([&](auto t_tag) {
      constexpr int t = decltype(t_tag)::value;
      unit(piece + t / PL, std::integral_constant<int, t / PL>{}, std::integral_constant<int, t % PL>{}, std::integral_constant<int, kMany>{});
    });
  int image[PL];                                 // the stage that takes plane q of the addend and of the output
  static_for<0, 2 * PL>([&](auto t_tag) {        // the last two pieces
    constexpr int t = decltype(t_tag)::value, left = 2 * PL - 1 - t;
    if constexpr (NST - 1 - left >= 0 && NST - 1 - left < PL) image[NST - 1 - left] = stage;
    unit(piece + t / PL, std::integral_constant<int, t / PL>{}, std::integral_constant<int, t % PL>{}, std::integral_constant<int, left>{});
  });
  wait_vmcnt<0>();
  __syncthreads();                               // every wave has read the last unit, and the addend is there

  // ---- epilogue: val = alpha * (beta_acc * acc + beta_e * sum of the addend's planes); plane q of the output is bf16(val_q)
  // with val_0 = val and val_{q+1} = val_q - bf16(val_q) (exact) ----
  const int el = thread_index(0), er = el & 31, eh = el >> 5;    // lane, as fr and fh: worked out anew, not kept through the loop
  const float ab_acc = alpha * beta_acc, ab_e = alpha * beta_e;
  u16* C = static_cast<u16*>(p.C);
  u16* Ct = static_cast<u16*>(p.Ct);
  int ldct = p.ldct;
  if (p.symmetric) {                             // mirror store; the tile itself only off the diagonal
    Ct = C;
    ldct = p.ldc;
    if (diagonal) C = nullptr;
  }
  auto slot = [&](int q, int row, int chunk) -> u32x2* {
    return reinterpret_cast<u32x2*>(smem + image[q] * UNIT_B + row * (2 * BT) + ((chunk ^ key(row)) * 16) + eh * 8);
  };
  auto pack2f = [](float x, float y) {
    const f32x2 v = {x, y};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
  };
  u32x2 pk[PL][F][F][4];
#pragma unroll
  for (int i = 0; i < F; ++i)
#pragma unroll
    for (int j = 0; j < F; ++j) {
      const int row = wn * WT + 32 * j + er, chunk0 = wm * (WT / 8) + 4 * i;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        float x[4] = {0.f, 0.f, 0.f, 0.f};       // smallest terms first: two of the sums are rounded at the size of the result
        auto add_plane = [&](int q) {
          const u32x2 e = *slot(q, row, chunk0 + k);
          x[0] = fmaf(ab_e, __uint_as_float(e.x << 16), x[0]);
          x[1] = fmaf(ab_e, __uint_as_float(e.x & 0xffff0000u), x[1]);
          x[2] = fmaf(ab_e, __uint_as_float(e.y << 16), x[2]);
          x[3] = fmaf(ab_e, __uint_as_float(e.y & 0xffff0000u), x[3]);
        };
        if constexpr (ADD) {
#pragma unroll
          for (int q = PL - 1; q > 0; --q) add_plane(q);
        }
        if constexpr (SPLIT) {
#pragma unroll
          for (int v = 0; v < 4; ++v) x[v] = fmaf(ab_acc, acc[2][i][j][4 * k + v], x[v]);
        }
        if constexpr (ADD) add_plane(0);
#pragma unroll
        for (int v = 0; v < 4; ++v) x[v] = fmaf(ab_acc, SPLIT ? acc[0][i][j][4 * k + v] + acc[SPLIT][i][j][4 * k + v] : acc[0][i][j][4 * k + v], x[v]);
#pragma unroll
        for (int q = 0; q < PL; ++q) {
          const u32x2 w = {pack2f(x[0], x[1]), pack2f(x[2], x[3])};
          pk[q][i][j][k] = w;
          x[0] -= __uint_as_float(w.x << 16);    // what this plane leaves of the value
          x[1] -= __uint_as_float(w.x & 0xffff0000u);
          x[2] -= __uint_as_float(w.y << 16);
          x[3] -= __uint_as_float(w.y & 0xffff0000u);
          *slot(q, row, chunk0 + k) = w;
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  // an image leaves with 16 bytes per lane
  auto store_images = [&](u16* dst, int64_t plane, int ld, int first_row, int first_col) {
    __syncthreads();
#pragma unroll
    for (int q = 0; q < PL; ++q) {
      u32x4 v[NIMG];
#pragma unroll
      for (int n = 0; n < NIMG; ++n)
        v[n] = *reinterpret_cast<const u32x4*>(smem + image[q] * UNIT_B + (n * NW + wave) * 1024 + el * 16);
#pragma unroll
      for (int n = 0; n < NIMG; ++n) {
        const int r = (n * NW + wave) * RPI + el / CPT;
        *(gvec_ptr)(dst + (size_t)q * (size_t)plane + (size_t)(first_row + r) * ld + first_col + ((el % CPT) ^ key(r)) * 8) = v[n];
      }
    }
  };
  if (Ct) store_images(Ct, p.symmetric ? p.c_plane : p.ct_plane, ldct, col0, row0);
  if (C) {                                       // the tile itself: through a transpose on the matrix cores (exact)
    bf16x8 sel[2];                               // 0/1 selector
#pragma unroll
    for (int sx = 0; sx < 2; ++sx)
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const int row = 16 * sx + 4 * eh + (t < 4 ? t : 4 + t);
        sel[sx][t] = (__bf16)(er == row ? 1.0f : 0.0f);
      }
    __syncthreads();                             // the images have been read out (or the addend has)
#pragma unroll
    for (int q = 0; q < PL; ++q)
#pragma unroll
      for (int i = 0; i < F; ++i)
#pragma unroll
        for (int j = 0; j < F; ++j) {
          f32x16 d;
#pragma unroll
          for (int v = 0; v < 16; ++v) d[v] = 0.f;
#pragma unroll
          for (int sx = 0; sx < 2; ++sx) {
            const u32x4 raw = {pk[q][i][j][2 * sx].x, pk[q][i][j][2 * sx].y, pk[q][i][j][2 * sx + 1].x, pk[q][i][j][2 * sx + 1].y};
            d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, raw), sel[sx], d, 0, 0, 0);
          }
#pragma unroll
          for (int k = 0; k < 4; ++k)
            *slot(q, wm * WT + 32 * i + er, wn * (WT / 8) + 4 * j + k) = u32x2{pack2f(d[4 * k], d[4 * k + 1]), pack2f(d[4 * k + 2], d[4 * k + 3])};
          __builtin_amdgcn_sched_barrier(0);
        }
    store_images(C, p.c_plane, p.ldc, row0, col0);
  }
}

// (the apply product, K-major, always has an addend: with planes the a X term is not folded into the polynomial)
template <int BT, int NST, bool LKM, int PL>
__device__ __forceinline__ void planes_tile(const GemmProblem& p, int row0, int col0, bool diagonal, unsigned char* smem,
                                            float beta_acc, float beta_e, int alpha_idx, double eps) {
  if (LKM || p.Et) gemm_planes_body<BT, NST, LKM, PL, true>(p, row0, col0, diagonal, smem, beta_acc, beta_e, alpha_idx, eps);
  else gemm_planes_body<BT, NST, LKM, PL, false>(p, row0, col0, diagonal, smem, beta_acc, beta_e, alpha_idx, eps);
}

}  // namespace
}  // namespace muon
