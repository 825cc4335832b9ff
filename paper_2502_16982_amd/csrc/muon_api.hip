// C ABI and host-side planner of the MI355X Muon step (see include/muon.h for the contract).
//
// muon_init turns a list of matrix shapes into: the orientation and padded extents of every matrix, the
// chunking of the list against the workspace, and device tables (matrix records, elementwise tiles, one
// grouped-GEMM problem table and tile table per Newton-Schulz product).  muon_step only enqueues kernels.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <new>
#include <vector>

#include "../../include/muon.h"
#include "muon_launch.h"
#include "muon_plan.h"

using namespace muon;

namespace {

thread_local int g_last_hip_error = 0;

inline int hip_fail(hipError_t e) {
  g_last_hip_error = (int)e;
  return MUON_E_HIP;
}
#define MUON_HIP(expr)                          \
  do {                                          \
    hipError_t e__ = (expr);                    \
    if (e__ != hipSuccess) return hip_fail(e__); \
  } while (0)

// Every entry point runs its body through this: nothing may unwind through the C ABI.
template <typename F>
int guarded(F&& body) noexcept {
  try {
    return body();
  } catch (const std::bad_alloc&) {
    return MUON_E_NO_MEMORY;
  } catch (...) {
    return MUON_E_INVALID_ARG;
  }
}

// Scratch of muon_step_static, the entry point for callers that cannot allocate device memory: the tables and
// Newton-Schulz temporaries that muon_step keeps in the caller's workspace live in this array instead.  Every device
// the library runs on holds its own copy, at its own address, until the process ends.  In host code the name is only
// a handle for hipGetSymbolAddress; the device address it yields (StaticSlot::ptr) is what kernels and copies get.
constexpr size_t kStaticScratchBytes = MUON_STATIC_MAX_BYTES;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

}  // namespace

namespace {

// One product of a group's sequence.
struct GroupOp {
  int product;        // PairProduct
  size_t probs;       // offset of the problem table
  float beta_acc, beta_e, diag_add;
  int alpha_idx, kind;
};

}  // namespace

struct muon_ctx {
  int n = 0;
  int ns_dtype = MUON_BF16;
  int device = 0;
  Plan plan;             // orientation, padding, chunking, host image of the device tables
  unsigned char* ws = nullptr;
  size_t ws_bytes = 0;
  // device tables
  MatDesc* d_mats = nullptr;
  MatPtrs* d_ptrs = nullptr;
  // dynamic pointer upload
  MatPtrs* h_ptrs_pinned = nullptr;
  std::vector<MatPtrs> last_ptrs;
  bool ptrs_valid = false;
  hipEvent_t upload_done = nullptr;
  // host-only plan (muon_plan_only): no device tables exist
  bool plan_only = false;
  // state of the last step, for the debug read
  int last_o_sel = 0, last_use_s = 0, last_chunk = -1;
  // scratch of a step, kept from step to step: coefficients of every iteration, products of the two groups
  std::vector<double> coeff;
  std::vector<GroupOp> group_ops[2];
  // optional per-launch event timing
  bool profiling = false;
  std::vector<hipEvent_t> prof_events;   // pairs: start, stop
  std::vector<int> prof_pending;         // kernel class of each pending pair
  double prof_ms[MUON_PROF_COUNT] = {};
  int64_t prof_launches[MUON_PROF_COUNT] = {};
};

namespace {

constexpr size_t kProfPairs = 2048;

int prof_drain(muon_ctx* ctx) {
  for (size_t i = 0; i < ctx->prof_pending.size(); ++i) {
    float ms = 0.f;
    MUON_HIP(hipEventSynchronize(ctx->prof_events[2 * i + 1]));
    MUON_HIP(hipEventElapsedTime(&ms, ctx->prof_events[2 * i], ctx->prof_events[2 * i + 1]));
    ctx->prof_ms[ctx->prof_pending[i]] += (double)ms;
    ctx->prof_launches[ctx->prof_pending[i]] += 1;
  }
  ctx->prof_pending.clear();
  return MUON_OK;
}

// Brackets one launch with events when profiling is on.
template <typename F>
int timed(muon_ctx* ctx, int cls, hipStream_t s, F&& launch) {
  if (!ctx->profiling) {
    MUON_HIP(launch());
    return MUON_OK;
  }
  if (ctx->prof_pending.size() >= kProfPairs) {
    int st = prof_drain(ctx);
    if (st != MUON_OK) return st;
  }
  const size_t k = ctx->prof_pending.size();
  MUON_HIP(hipEventRecord(ctx->prof_events[2 * k], s));
  MUON_HIP(launch());
  MUON_HIP(hipEventRecord(ctx->prof_events[2 * k + 1], s));
  ctx->prof_pending.push_back(cls);
  return MUON_OK;
}
#define MUON_TIMED(cls, call)                                   \
  do {                                                          \
    int st__ = timed(ctx, cls, s, [&]() { return (call); });    \
    if (st__ != MUON_OK) return st__;                           \
  } while (0)

}  // namespace

extern "C" {

int muon_default_hparams(muon_hparams* hp) {
  if (!hp) return MUON_E_INVALID_ARG;
  hp->lr = 0.0;
  hp->weight_decay = 0.0;
  hp->momentum = 0.95;
  hp->a = 3.4445;
  hp->b = -4.7750;
  hp->c = 2.0315;
  hp->rms_scale = 0.2;
  hp->eps = 1e-7;
  hp->ns_steps = 5;
  hp->nesterov = 1;
  hp->scale_mode = MUON_SCALE_ADJUSTED_LR;
  hp->reserved = 0;
  hp->hidden_size = 0.0;
  hp->coeff_schedule = nullptr;
  return MUON_OK;
}

int muon_workspace_bytes(const muon_param* shapes, int32_t n, int32_t ns_dtype, size_t max_bytes, size_t* out) {
  return guarded([&]() { return plan_workspace_bytes(shapes, n, ns_dtype, max_bytes, out); });
}

}  // extern "C"

namespace {

// Validates the arguments of a step against the plan.  *changed: the pointer list differs from the uploaded one.
int check_step_args(const muon_ctx* ctx, const muon_param* params, int32_t n, const muon_hparams* hp, bool* changed) {
  if (!ctx || !params || !hp || ctx->plan_only) return MUON_E_INVALID_ARG;
  if (n != ctx->n) return MUON_E_SHAPE_MISMATCH;
  if (hp->ns_steps < 0 || !(hp->eps >= 0.0) || !std::isfinite(hp->lr) || !std::isfinite(hp->weight_decay) ||
      !std::isfinite(hp->momentum) || !std::isfinite(hp->a) || !std::isfinite(hp->b) || !std::isfinite(hp->c) ||
      !std::isfinite(hp->rms_scale) || hp->scale_mode < MUON_SCALE_ADJUSTED_LR || hp->scale_mode > MUON_SCALE_UPDATE_NORM ||
      hp->reserved != 0 || (hp->scale_mode == MUON_SCALE_BASELINE && !(hp->hidden_size > 0.0 && std::isfinite(hp->hidden_size))))
    return MUON_E_INVALID_ARG;
  if (hp->coeff_schedule)
    for (int i = 0; i < 3 * hp->ns_steps; ++i)
      if (!std::isfinite(hp->coeff_schedule[i])) return MUON_E_INVALID_ARG;
  *changed = !ctx->ptrs_valid;
  for (int i = 0; i < n; ++i) {
    const muon_param& p = params[i];
    const MatPlan& q = ctx->plan.mats[i];
    if (p.rows != q.rows || p.cols != q.cols || p.w_dtype != q.w_dtype || p.g_dtype != q.g_dtype) return MUON_E_SHAPE_MISMATCH;
    if (!p.w || !p.g || !p.m) return MUON_E_INVALID_ARG;
    const uintptr_t wa = p.w_dtype == MUON_BF16 ? 1u : 3u, ga = p.g_dtype == MUON_BF16 ? 1u : 3u;
    if ((reinterpret_cast<uintptr_t>(p.w) & wa) || (reinterpret_cast<uintptr_t>(p.g) & ga) || (reinterpret_cast<uintptr_t>(p.m) & 3u))
      return MUON_E_MISALIGNED;
    const MatPtrs& l = ctx->last_ptrs[i];
    if (l.w != p.w || l.g != p.g || l.m != p.m) *changed = true;
  }
  return MUON_OK;
}

int quarter_flags(bool quarters, int few) {
  return !quarters && few == 3 ? kGemmRing128 : quarters ? kGemmQuarters | (few == 2 ? kGemmSixteenths : few == 1 ? kGemmFewQuarters : 0) : 0;
}

// The products of a group's N iterations, in order.  coeff: a, b, c of every iteration.
void list_ops(const Group& g, int N, const double* coeff, bool gram, bool fold, std::vector<GroupOp>& out) {
  out.clear();
  if (g.n_prob == 0) return;
  const int norm = fold ? kAlphaFromPartials : 1;
  if (!gram) {
    for (int it = 0; it < N; ++it) {
      const int first = it == 0, last = it == N - 1, par = it & 1;
      const float a = (float)coeff[3 * it], b = (float)coeff[3 * it + 1], c = (float)coeff[3 * it + 2];
      out.push_back({kPairGram, g.prob_gram[par], 1.f, 0.f, 0.f, first ? norm : -1, 0});
      out.push_back({kPairSym, g.prob_poly, c, b, a, -1, 0});
      out.push_back({kPairApply, g.prob_apply[par * 2 + last], 1.f, a, 0.f, first ? 0 : -1, kSideKMajor});
    }
    return;
  }
  // the Gram route (muon_plan.h); its scales are powers of two and change nothing but exponents
  const float SA = kGramScaleA, SP = kGramScaleP, SX = kGramScaleX;
  const int f16 = kSideInF16 | kSideOutF16;
  int par = 0;
  for (int it = 0; it < N; par ^= 1) {
    const int steps = gram_group(it, N);
    const bool first = it == 0, last = it + steps == N;
    auto op = [&](int o) { return g.prob_ops + sizeof(GemmProblem) * (size_t)g.n_prob * (size_t)(o < kGramParityOps ? par * kGramParityOps + o : o); };
    float a = (float)coeff[3 * it], b = (float)coeff[3 * it + 1], c = (float)coeff[3 * it + 2];
    if (first) {                     // U, in bf16: as it is written
      out.push_back({kPairGram, g.prob_gram[par], 1.f, 0.f, 0.f, norm, 0});
      out.push_back({kPairSym, g.prob_poly, c, b, a, -1, 0});
    } else {
      out.push_back({kPairGram, g.prob_gram[par], SA / (SX * SX), 0.f, 0.f, 2, f16});           // (alphas: store_norm)
      out.push_back({kPairSym, g.prob_poly, c * (SP / (SA * SA)), b * (SP / SA), a * SP, -1, f16});
    }
    if (steps == 2) {
      const double* k = coeff + 3 * (it + 1);
      a = (float)k[0], b = (float)k[1], c = (float)k[2];
      out.push_back({kPairSym, op(kGramT), 1.f / SP, 0.f, 0.f, -1, f16});
      out.push_back({kPairSym, op(kGramA), 1.f / SP, 0.f, 0.f, -1, f16});
      out.push_back({kPairSym, op(kGramD), c * (SP / (SA * SA)), b * (SP / SA), 0.f, -1, f16});
      out.push_back({kPairSym, op(kGramQ), 1.f / SP, a, 0.f, -1, f16});
    }
    it += steps;
    out.push_back({kPairApply, steps == 2 ? op(kGramApply + par * 2 + last) : g.prob_apply[par * 2 + last], (last ? 1.f : SX) / (first ? 1.f : SP * SX),
                   0.f, 0.f, first ? 0 : last ? 3 : -1, kSideKMajor | (first ? 0 : kSideInF16) | (last ? 0 : kSideOutF16)});
  }
}

// Iterations of a chunk with matrices of the Gram route: the next product of either group in every launch.
int enqueue_paired(muon_ctx* ctx, const Chunk& ch, const muon_hparams* hp, const double* coeff, bool gram, float gain, bool fold, hipStream_t s) {
  std::vector<GroupOp>* const ops = ctx->group_ops;
  for (int i = 0; i < 2; ++i) list_ops(ch.groups[i], hp->ns_steps, coeff, i == 1 && gram, fold, ops[i]);
  size_t at[2] = {0, 0};
  while (at[0] < ops[0].size() || at[1] < ops[1].size()) {
    const GroupOp* op[2];
    for (int i = 0; i < 2; ++i) op[i] = at[i] < ops[i].size() ? &ops[i][at[i]] : nullptr;
    // An apply product in coarse tiles shares its launch with a product of the other group that is all fine tiles and not too many.
    // Otherwise it runs alone and a symmetric product of the other group waits for the next one of this.
    // Two apply products that read bf16, the first iteration's, have a table of both where that saves a round.
    const bool joint = op[0] && op[1] && op[0]->product == kPairApply && op[1]->product == kPairApply && ch.n_shared_app > 0 &&
                       !((op[0]->kind | op[1]->kind) & kSideInF16);
    int applied = -1;                // group of that apply product
    bool beside = false;
    for (int i = 0; i < 2 && op[0] && op[1] && applied < 0 && !joint; ++i)
      if (op[i]->product == kPairApply && ch.groups[i].coarse.n_apply > 0) {
        beside = ch.beside[i ^ 1][op[i ^ 1]->product];
        if (beside || op[i ^ 1]->product != kPairApply) applied = i;
      }
    for (int i = 0; i < 2; ++i) {
      if (applied >= 0 && i != applied && !beside) op[i] = nullptr;
      at[i] += op[i] ? 1 : 0;
    }
    const int product[2] = {op[0] ? op[0]->product : kPairNone, op[1] ? op[1]->product : kPairNone};
    const PairForm& form = ch.pair[product[0]][product[1]];
    const int timed_as = product[1] == kPairApply || product[0] == kPairApply ? MUON_PROF_APPLY_POLY
                         : product[1] == kPairGram || product[0] == kPairGram ? MUON_PROF_GRAM : MUON_PROF_POLY;
    // a symmetric product with too few coarse tiles and no other beside it: all of it in the fine launch
    const bool lone = op[1] && product[1] == kPairSym && ch.groups[1].n_lone > 0 && (!op[0] || product[0] == kPairApply);
    const bool both_sym = op[0] && op[1] && product[0] != kPairApply && product[1] != kPairApply;
    for (int level = lone && !beside ? 0 : 1; level >= 0; --level) {
      GemmSide side[2] = {};
      int64_t longest[2] = {0, 0};
      bool strips = false;
      for (int i = 0; i < 2; ++i) {
        side[i].alpha_idx = -1;
        const bool guest = beside && i != applied;            // all of it in the coarse launch
        const Group& g = ch.groups[i];
        if (!op[i] || (guest && level == 0) || (joint && level == 0 && g.coarse.n_apply == 0)) continue;
        const TileSet& ts = level && !guest ? g.coarse : g.fine;
        const bool gram_product = product[i] == kPairGram, apply = product[i] == kPairApply;
        const bool from_lone = lone && i == 1;
        side[i].n_tiles = joint && level ? ch.n_shared_app : from_lone ? g.n_lone : gram_product ? ts.n_sym : apply ? ts.n_apply : ts.n_poly;
        if (side[i].n_tiles == 0) continue;
        side[i].tiles = reinterpret_cast<const GemmTile*>(ctx->ws + (from_lone ? g.lone : gram_product ? ts.sym : apply ? ts.apply : ts.poly));
        side[i].probs = reinterpret_cast<const GemmProblem*>(ctx->ws + op[i]->probs);
        side[i].beta_acc = op[i]->beta_acc;
        side[i].beta_e = op[i]->beta_e;
        side[i].diag_add = op[i]->diag_add;
        side[i].alpha_idx = op[i]->alpha_idx;
        side[i].kind = op[i]->kind;
        side[i].gain = i == 1 ? gain : 0.f;
        longest[i] = gram_product ? g.longest_n : g.longest_m;
        strips = strips || ts.strips;
      }
      if (side[0].n_tiles + side[1].n_tiles == 0) continue;
      const auto own = [&](int i) { return ch.groups[i].coarse.n_apply > 0 ? kPairApply : kPairNone; };
      const PairForm& fine_form = joint ? ch.pair[own(0)][own(1)] : beside ? ch.pair[applied == 0 ? kPairApply : kPairNone][applied == 1 ? kPairApply : kPairNone]
                                  : lone ? ch.groups[1].lone_form[op[0] != nullptr] : form;
      const int flags = level ? (strips ? kGemmStrips : 0) | (form.persistent ? kGemmPersistent : 0) : quarter_flags(fine_form.quarters, fine_form.few);
      if (level && both_sym && ch.n_shared_sym > 0) {
        const size_t tiles = ch.shared_sym[product[0] != kPairGram][product[1] != kPairGram];
        MUON_TIMED(timed_as, launch_gemm_shared(flags, side[0], side[1], reinterpret_cast<const GemmTile*>(ctx->ws + tiles), ch.n_shared_sym, s));
        continue;
      }
      if (level && joint) {
        const int joint_flags = (ch.shared_app_strips ? kGemmStrips : 0) | (ch.shared_app_steady ? kGemmPersistent : 0);
        MUON_TIMED(timed_as, launch_gemm_shared(joint_flags, side[0], side[1], reinterpret_cast<const GemmTile*>(ctx->ws + ch.shared_app), ch.n_shared_app, s));
        continue;
      }
      if (level && beside) {
        MUON_TIMED(timed_as, launch_gemm_beside(flags, side[applied], side[applied ^ 1], s));
        continue;
      }
      const int x = longest[1] > longest[0];     // the longer K loops start first
      if (level) {                               // a launch for each
        for (int i : {x, x ^ 1})
          if (side[i].n_tiles > 0) MUON_TIMED(timed_as, launch_gemm_pair(1, flags, side[i], GemmSide{}, hp->eps, s));
        continue;
      }
      MUON_TIMED(timed_as, launch_gemm_pair(0, flags, side[x], side[x ^ 1], hp->eps, s));
    }
  }
  return MUON_OK;
}

// Enqueues every kernel of one step on stream s.  The pointer table is already on its way on the same stream, or (pack, plans
// of one chunk) the first pass takes the pointers as an argument and fills it.
int enqueue_step(muon_ctx* ctx, const muon_hparams* hp, hipStream_t s, float* update_rms_out, const PtrPack* pack = nullptr) {
  const int N = hp->ns_steps;
  const int use_s = N == 0;
  const bool mc = on_matrix_cores(ctx->ns_dtype);   // bf16 or split-bf16: the MFMA kernels and their one-layout plan
  const int planes = planes_of(ctx->ns_dtype);
  // where O ends up (see o_source in the elementwise kernels): fp32 path: X in place, its transpose in Xt[N & 1];
  // bf16 path: X ping-pong index N & 1 (bit 1), transposed matrices in Xt[1], or Xt[0] when no iteration ran (bit 0)
  const int o_written = mc ? ((N & 1) << 1) | (N > 0 ? 1 : 0) : (N & 1);
  std::vector<double>& coeff = ctx->coeff;
  double gain = 0.0;
  bool gram = false;                 // (lists without matrices of the Gram route spend no host time on its coefficients)
  for (const Chunk& ch : ctx->plan.chunks) gram = gram || ch.paired;
  if (gram) {
    coeff.resize(3 * (size_t)N);
    for (int i = 0; i < 3 * N; ++i) coeff[i] = hp->coeff_schedule ? hp->coeff_schedule[i] : i % 3 == 0 ? hp->a : i % 3 == 1 ? hp->b : hp->c;
    gram = N >= kGramMinSteps && gram_coefficients_fit(coeff.data(), N, &gain);
  }
  const float gram_gain = gram ? (float)gain : 0.f;
  const int o_sel = o_written | (gram ? (gram_groups(N) & 1) << 1 | 1 : o_written) << 2;

  for (size_t ci = 0; ci < ctx->plan.chunks.size(); ++ci) {
    const Chunk& ch = ctx->plan.chunks[ci];
    const EwTile* ew = reinterpret_cast<const EwTile*>(ctx->ws + ch.ew_tiles_off);
    MUON_TIMED(MUON_PROF_MOMENTUM, launch_momentum_norm_cast(ctx->d_mats, ctx->d_ptrs, pack, ew, ch.n_ew_tiles, (float)hp->momentum,
                                                             hp->nesterov != 0, (!mc || N == 0) ? 1 : 0, ctx->ns_dtype, s));
    const bool fold = ch.fold_norm && N > 0;
    if (!fold) MUON_TIMED(MUON_PROF_NORM, launch_norm_finalize(ctx->d_mats, ch.first, ch.count, hp->eps, gram_gain, s));
    if (ch.paired) {
      const int st = enqueue_paired(ctx, ch, hp, coeff.data(), gram, gram_gain, fold, s);
      if (st != MUON_OK) return st;
    }
    for (int it = 0; it < N && !ch.paired; ++it) {
      const int first = it == 0, last = it == N - 1, par = it & 1;
      const double* sch = hp->coeff_schedule ? hp->coeff_schedule + 3 * it : nullptr;
      const float a = (float)(sch ? sch[0] : hp->a), b = (float)(sch ? sch[1] : hp->b), c = (float)(sch ? sch[2] : hp->c);
      for (const Group& g : ch.groups) {
        auto P = [&](size_t o) { return reinterpret_cast<const GemmProblem*>(ctx->ws + o); };
        auto T = [&](size_t o) { return reinterpret_cast<const GemmTile*>(ctx->ws + o); };
        // one launch per product and level (the coarse tiles first, then what they leave)
        for (int level = 1; level >= 0; --level) {
          const TileSet& ts = level ? g.coarse : g.fine;
          if (ts.n_sym == 0) continue;
          if (mc)
            MUON_TIMED(MUON_PROF_GRAM, launch_gemm_bf16(level, (ts.strips ? kGemmStrips : 0) | (ts.persistent_n ? kGemmPersistent : 0) | quarter_flags(ts.quarter_sym, ts.few_sym), P(g.prob_gram[par]), T(ts.sym), ts.n_sym, 1.f, 0.f,
                                                        first ? (fold ? kAlphaFromPartials : 1) : -1, hp->eps, 0.f, 0, planes, s));
          else
            MUON_TIMED(MUON_PROF_GRAM, launch_gemm_f32((ts.quarter_sym ? kGemmQuarters : 0) | (ts.long_n ? kGemmLongK : 0), ts.tail_sym, P(g.prob_gram[par]), T(ts.sym), ts.n_sym, 1.f, 0.f,
                                                       first ? (fold ? kAlphaFromPartials : 1) : -1, hp->eps, s));
        }
        for (int level = 1; level >= 0; --level) {
          const TileSet& ts = level ? g.coarse : g.fine;
          if (ts.n_poly == 0) continue;
          if (mc)
            MUON_TIMED(MUON_PROF_POLY, launch_gemm_bf16(level, (ts.strips ? kGemmStrips : 0) | (ts.persistent_m ? kGemmPersistent : 0) | quarter_flags(ts.quarter_poly, ts.few_poly), P(g.prob_poly), T(ts.poly), ts.n_poly, c, b, -1, 0.0, a, 0, planes, s));
          else
            MUON_TIMED(MUON_PROF_POLY, launch_gemm_f32((ts.quarter_poly ? kGemmQuarters : 0) | (ts.long_m ? kGemmLongK : 0), ts.tail_poly, P(g.prob_poly), T(ts.poly), ts.n_poly, c, b, -1, 0.0, s));
        }
        for (int level = 1; level >= 0; --level) {
          const TileSet& ts = level ? g.coarse : g.fine;
          if (ts.n_apply == 0) continue;
          if (mc)
            MUON_TIMED(MUON_PROF_APPLY_POLY, launch_gemm_bf16(level, (ts.strips ? kGemmStrips : 0) | (ts.persistent_m ? kGemmPersistent : 0) | quarter_flags(ts.quarter_apply, ts.few_apply), P(g.prob_apply[par * 2 + last]), T(ts.apply),
                                                              ts.n_apply, 1.f, a, first ? 0 : -1, 0.0, 0.f, 1, planes, s));
          else
            MUON_TIMED(MUON_PROF_APPLY_POLY, launch_gemm_f32((ts.quarter_apply ? kGemmQuarters : 0) | (ts.long_m ? kGemmLongK : 0), ts.tail_apply, P(g.prob_apply[par * 2 + last]), T(ts.apply), ts.n_apply, 1.f, a,
                                                             first ? 0 : -1, 0.0, s));
        }
      }
    }
    if (hp->scale_mode == MUON_SCALE_UPDATE_NORM) {
      // Eq. 6 needs RMS(O) before the update: one extra pass over O
      MUON_TIMED(MUON_PROF_RMS, launch_update_sumsq(ctx->d_mats, ew, ch.n_ew_tiles, o_sel, ctx->ns_dtype, s));
      MUON_TIMED(MUON_PROF_RMS, launch_update_rms(ctx->d_mats, ch.first, ch.count, use_s, 1, nullptr, s));
    }
    MUON_TIMED(MUON_PROF_UPDATE, launch_apply_update(ctx->d_mats, ctx->d_ptrs, ew, ch.n_ew_tiles, (float)hp->lr,
                                                     (float)hp->weight_decay, (float)hp->rms_scale, hp->scale_mode,
                                                     (float)std::sqrt(hp->hidden_size > 0.0 ? hp->hidden_size : 0.0), o_sel, use_s,
                                                     ch.stream_w, ctx->ns_dtype, s));
    if (update_rms_out) MUON_TIMED(MUON_PROF_RMS, launch_update_rms(ctx->d_mats, ch.first, ch.count, use_s, 0, update_rms_out, s));
  }
  ctx->last_o_sel = o_sel;
  ctx->last_use_s = use_s;
  ctx->last_chunk = (int)ctx->plan.chunks.size() - 1;
  return MUON_OK;
}

int step_impl(muon_ctx* ctx, const muon_param* params, int32_t n, const muon_hparams* hp, void* hip_stream,
              float* update_rms_out) {
  bool changed = false;
  const int st = check_step_args(ctx, params, n, hp, &changed);
  if (st != MUON_OK) return st;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  if (changed) {
    // the previous upload may still be reading the pinned staging buffer
    if (ctx->ptrs_valid) MUON_HIP(hipEventSynchronize(ctx->upload_done));
    // until the new table is known to be on its way, the device table counts as unknown: a failure below must not
    // leave a later step believing that its (identical) pointers are already uploaded
    ctx->ptrs_valid = false;
    for (int i = 0; i < n; ++i) ctx->h_ptrs_pinned[i] = MatPtrs{params[i].w, params[i].g, params[i].m};
    MUON_HIP(hipMemcpyAsync(ctx->d_ptrs, ctx->h_ptrs_pinned, sizeof(MatPtrs) * (size_t)n, hipMemcpyHostToDevice, s));
    MUON_HIP(hipEventRecord(ctx->upload_done, s));
    for (int i = 0; i < n; ++i) ctx->last_ptrs[i] = ctx->h_ptrs_pinned[i];
    ctx->ptrs_valid = true;
  }
  return enqueue_step(ctx, hp, s, update_rms_out);
}

}  // namespace

namespace {

// Everything muon_init does: the plan (host only) and, with `upload`, the transfer of its table image to the
// workspace and the per-context HIP objects.
int build_context(muon_ctx** out, const muon_param* shapes, int32_t n, int32_t ns_dtype, void* workspace,
                  size_t workspace_bytes, bool upload) {
  if (!out) return MUON_E_INVALID_ARG;
  *out = nullptr;
  int st = validate_shapes(shapes, n, ns_dtype);
  if (st != MUON_OK) return st;
  if (!workspace) return MUON_E_INVALID_ARG;
  if (reinterpret_cast<uintptr_t>(workspace) & 255u) return MUON_E_MISALIGNED;
  muon_ctx* ctx = new muon_ctx();
  struct Guard {     // releases the half-built context on every early return and on exceptions
    muon_ctx* c;
    ~Guard() { if (c) muon_destroy(c); }
  } guard{ctx};
  ctx->n = n;
  ctx->ns_dtype = ns_dtype;
  ctx->ws = static_cast<unsigned char*>(workspace);
  ctx->ws_bytes = workspace_bytes;
  {
    size_t least = 0;                // rejected before the device is touched
    st = plan_workspace_bytes(shapes, n, ns_dtype, 1, &least);
    if (st != MUON_OK) return st;
    if (workspace_bytes < least) return MUON_E_WORKSPACE_TOO_SMALL;
  }
  if (upload) {
    // before the plan: it evens out the persistent launches against the device's number of compute units
    hipError_t e = hipGetDevice(&ctx->device);
    if (e == hipSuccess) e = gemm_setup();
    if (e != hipSuccess) return hip_fail(e);
    ctx->plan.coarse_blocks = gemm_coarse_blocks();
  }
  st = plan_build(ctx->plan, shapes, n, ns_dtype, reinterpret_cast<uintptr_t>(workspace), workspace_bytes);
  if (st != MUON_OK) return st;
  ctx->d_mats = reinterpret_cast<MatDesc*>(ctx->ws + ctx->plan.off_mats);
  ctx->d_ptrs = reinterpret_cast<MatPtrs*>(ctx->ws + ctx->plan.off_ptrs);
  if (!upload) {
    ctx->plan_only = true;
  } else {
    hipError_t e = hipMemcpy(ctx->ws, ctx->plan.image.data(), ctx->plan.image.size(), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipHostMalloc(reinterpret_cast<void**>(&ctx->h_ptrs_pinned), sizeof(MatPtrs) * (size_t)n, hipHostMallocDefault);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&ctx->upload_done, hipEventDisableTiming);
    if (e != hipSuccess) return hip_fail(e);
    ctx->last_ptrs.resize(n);
  }
  guard.c = nullptr;
  *out = ctx;
  return MUON_OK;
}

}  // namespace

extern "C" {

int muon_init(muon_ctx** out, const muon_param* shapes, int32_t n, int32_t ns_dtype, void* workspace,
              size_t workspace_bytes) {
  return guarded([&]() { return build_context(out, shapes, n, ns_dtype, workspace, workspace_bytes, true); });
}

int muon_plan_only(muon_ctx** out, const muon_param* shapes, int32_t n, int32_t ns_dtype, size_t workspace_bytes) {
  // table pointers are computed from the workspace address but never followed: any aligned non-null address will do
  return guarded([&]() {
    return build_context(out, shapes, n, ns_dtype, reinterpret_cast<void*>(uintptr_t{1} << 32), workspace_bytes, false);
  });
}

int muon_plan_tiles(const muon_ctx* ctx, int32_t chunk, int32_t product, int32_t level, int32_t* out, int32_t cap_records) {
  if (!ctx || !ctx->plan_only || chunk < 0 || chunk >= (int)ctx->plan.chunks.size() || product < 0 || product > 3 || level < 0 ||
      level > 1 || cap_records < 0 || (cap_records > 0 && !out))
    return MUON_E_INVALID_ARG;
  return guarded([&]() { return (int)std::min<int64_t>(plan_tiles(ctx->plan, chunk, product, level, out, cap_records), INT32_MAX); });
}

int muon_step(muon_ctx* ctx, const muon_param* params, int32_t n, const muon_hparams* hp, void* hip_stream,
              float* update_rms_out) {
  return guarded([&]() { return step_impl(ctx, params, n, hp, hip_stream, update_rms_out); });
}

}  // extern "C"

namespace {

constexpr int kStaticMaxDevices = 64;
static_assert(kPackSlots == MUON_STATIC_MAX_MATRICES, "the per-step pointers of muon_step_static travel as a kernel argument");
struct StaticSlot {
  unsigned char* ptr = nullptr;      // device address of `scratch` on this device (hipGetSymbolAddress)
  muon_ctx* ctx = nullptr;           // plan and tables of the shape list of the last call on this device
  std::vector<muon_param> key;       // that shape list (rows, cols, dtypes)
};
StaticSlot g_static[kStaticMaxDevices];

int step_static_impl(const muon_param* params, int32_t n, int32_t ns_dtype, const muon_hparams* hp, void* hip_stream,
                     float* update_rms_out) {
  int st = validate_shapes(params, n, ns_dtype);
  if (st != MUON_OK) return st;
  if (!hp) return MUON_E_INVALID_ARG;
  if (n > MUON_STATIC_MAX_MATRICES) return MUON_E_STATIC_LIMIT;
  size_t need = 0;
  st = plan_workspace_bytes(params, n, ns_dtype, 0, &need);
  if (st != MUON_OK) return st;
  if (need > kStaticScratchBytes) return MUON_E_STATIC_LIMIT;

  int dev = 0;
  MUON_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kStaticMaxDevices) return MUON_E_INVALID_ARG;
  StaticSlot& slot = g_static[dev];
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  if (!slot.ptr) {                   // first call on this device: where does this device keep the array?
    void* p = nullptr;
    MUON_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p || (reinterpret_cast<uintptr_t>(p) & 255u)) return MUON_E_MISALIGNED;
    MUON_HIP(gemm_setup());
    slot.ptr = static_cast<unsigned char*>(p);
  }
  bool same = slot.ctx && slot.ctx->ns_dtype == ns_dtype && (int)slot.key.size() == n;
  for (int i = 0; same && i < n; ++i)
    same = slot.key[i].rows == params[i].rows && slot.key[i].cols == params[i].cols &&
           slot.key[i].w_dtype == params[i].w_dtype && slot.key[i].g_dtype == params[i].g_dtype;
  if (!same) {
    // Another shape list than the last call's: plan again (host memory only) and put the new tables at the head of
    // the scratch.  Earlier work on this stream may still be using the old tables, and the copy reads host memory
    // that must outlive it: wait on both sides of it.  The array keeps whatever the last call left; nothing in it has
    // to start at zero (every temporary is written in full before it is read), only the tables must be the new ones.
    MUON_HIP(hipStreamSynchronize(s));
    if (slot.ctx) {
      muon_destroy(slot.ctx);
      slot.ctx = nullptr;
    }
    muon_ctx* ctx = new muon_ctx();
    struct Guard {
      muon_ctx* c;
      ~Guard() { if (c) muon_destroy(c); }
    } guard{ctx};
    ctx->n = n;
    ctx->ns_dtype = ns_dtype;
    ctx->device = dev;
    ctx->ws = slot.ptr;
    ctx->ws_bytes = kStaticScratchBytes;
    ctx->plan.coarse_blocks = gemm_coarse_blocks();
    st = plan_build(ctx->plan, params, n, ns_dtype, reinterpret_cast<uintptr_t>(slot.ptr), kStaticScratchBytes);
    if (st != MUON_OK) return st;
    if (ctx->plan.chunks.size() != 1) return MUON_E_STATIC_LIMIT;
    ctx->d_mats = reinterpret_cast<MatDesc*>(ctx->ws + ctx->plan.off_mats);
    ctx->d_ptrs = reinterpret_cast<MatPtrs*>(ctx->ws + ctx->plan.off_ptrs);
    ctx->last_ptrs.resize(n);
    MUON_HIP(hipMemcpyAsync(slot.ptr, ctx->plan.image.data(), ctx->plan.image.size(), hipMemcpyHostToDevice, s));
    MUON_HIP(hipStreamSynchronize(s));
    slot.key.assign(params, params + n);
    slot.ctx = ctx;
    guard.c = nullptr;
  }
  muon_ctx* ctx = slot.ctx;
  ctx->ptrs_valid = true;            // check_step_args compares against last_ptrs only to report a change; unused here
  bool changed = false;
  st = check_step_args(ctx, params, n, hp, &changed);
  if (st != MUON_OK) return st;
  PtrPack pack{};
  for (int i = 0; i < n; ++i) pack.p[i] = MatPtrs{params[i].w, params[i].g, params[i].m};
  return enqueue_step(ctx, hp, s, update_rms_out, &pack);
}

}  // namespace

extern "C" {

int muon_step_static(const muon_param* params, int32_t n, int32_t ns_dtype, const muon_hparams* hp, void* hip_stream,
                     float* update_rms_out) {
  return guarded([&]() { return step_static_impl(params, n, ns_dtype, hp, hip_stream, update_rms_out); });
}

int muon_debug_read_update(muon_ctx* ctx, int32_t index, void* dst, int32_t dst_dtype, void* hip_stream) {
  if (!ctx || ctx->plan_only || !dst || index < 0 || index >= ctx->n) return MUON_E_INVALID_ARG;
  if (dst_dtype != MUON_F32 && dst_dtype != MUON_BF16) return MUON_E_UNSUPPORTED_DTYPE;
  if (ctx->last_chunk < 0 || ctx->plan.mats[index].chunk != ctx->last_chunk) return MUON_E_NOT_RESIDENT;
  MUON_HIP(launch_read_update(ctx->d_mats, index, ctx->last_o_sel, ctx->last_use_s, ctx->ns_dtype, dst, dst_dtype,
                              static_cast<hipStream_t>(hip_stream)));
  return MUON_OK;
}

int muon_plan_describe(const muon_ctx* ctx, int32_t index, int64_t* out, int32_t cap) {
  if (!ctx || !out || index < 0 || index >= ctx->n || cap < 0) return MUON_E_INVALID_ARG;
  const MatPlan& q = ctx->plan.mats[index];
  const int64_t v[9] = {q.m, q.n, q.transposed, q.mp, q.np, q.chunk, q.coarse ? kCoarse : q.tile, q.tile, q.gram};
  const int k = std::min<int>(cap, 9);
  for (int i = 0; i < k; ++i) out[i] = v[i];
  return k;
}

int muon_profile_enable(muon_ctx* ctx, int enable) {
  if (!ctx || ctx->plan_only) return MUON_E_INVALID_ARG;
  return guarded([&]() -> int {
  if (enable && ctx->prof_events.empty()) {
    ctx->prof_events.reserve(2 * kProfPairs);
    for (size_t i = 0; i < 2 * kProfPairs; ++i) {
      hipEvent_t ev = nullptr;
      MUON_HIP(hipEventCreate(&ev));
      ctx->prof_events.push_back(ev);
    }
  }
  if (!enable && ctx->profiling) {
    int st = prof_drain(ctx);
    if (st != MUON_OK) return st;
  }
  ctx->profiling = enable != 0;
  return MUON_OK;
  });
}

int muon_profile_read(muon_ctx* ctx, double* ms_out, int64_t* launches_out, int reset) {
  if (!ctx) return MUON_E_INVALID_ARG;
  int st = prof_drain(ctx);
  if (st != MUON_OK) return st;
  for (int i = 0; i < MUON_PROF_COUNT; ++i) {
    if (ms_out) ms_out[i] = ctx->prof_ms[i];
    if (launches_out) launches_out[i] = ctx->prof_launches[i];
    if (reset) {
      ctx->prof_ms[i] = 0.0;
      ctx->prof_launches[i] = 0;
    }
  }
  return MUON_OK;
}

int muon_adamw_step(const muon_adamw_param* params, int32_t n, const muon_adamw_hparams* hp, void* hip_stream) {
  if (!params || !hp || n <= 0) return MUON_E_INVALID_ARG;
  if (!(hp->beta1 >= 0.0 && hp->beta1 < 1.0) || !(hp->beta2 >= 0.0 && hp->beta2 < 1.0) || !(hp->eps >= 0.0) || hp->step < 1 ||
      !std::isfinite(hp->lr) || !std::isfinite(hp->weight_decay) || !std::isfinite(hp->eps))
    return MUON_E_INVALID_ARG;
  for (int i = 0; i < n; ++i) {
    const muon_adamw_param& q = params[i];
    if (!q.p || !q.g || !q.m || !q.v || q.numel < 1) return MUON_E_INVALID_ARG;
    if ((q.p_dtype != MUON_F32 && q.p_dtype != MUON_BF16) || (q.g_dtype != MUON_F32 && q.g_dtype != MUON_BF16))
      return MUON_E_UNSUPPORTED_DTYPE;
    const uintptr_t pa = q.p_dtype == MUON_BF16 ? 1u : 3u, ga = q.g_dtype == MUON_BF16 ? 1u : 3u;
    if ((reinterpret_cast<uintptr_t>(q.p) & pa) || (reinterpret_cast<uintptr_t>(q.g) & ga) ||
        (reinterpret_cast<uintptr_t>(q.m) & 3u) || (reinterpret_cast<uintptr_t>(q.v) & 3u))
      return MUON_E_MISALIGNED;
    if (q.numel > kAdamwMaxNumel) return MUON_E_INVALID_ARG;
  }
  // bias corrections in double, handed to the kernel as reciprocals
  const float inv_bc1 = (float)(1.0 / (1.0 - std::pow(hp->beta1, (double)hp->step)));
  const float inv_bc2 = (float)(1.0 / (1.0 - std::pow(hp->beta2, (double)hp->step)));
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  AdamwBatch b{};
  AdamwCursor at;
  while (const int blocks = adamw_next_batch(params, n, at, b))
    MUON_HIP(launch_adamw(b, blocks, (float)hp->lr, (float)hp->weight_decay, (float)hp->beta1, (float)hp->beta2, (float)hp->eps,
                          inv_bc1, inv_bc2, s));
  return MUON_OK;
}

int muon_plan_chunks(const muon_ctx* ctx) { return ctx ? (int)ctx->plan.chunks.size() : MUON_E_INVALID_ARG; }

void muon_destroy(muon_ctx* ctx) {
  if (!ctx) return;
  if (ctx->upload_done) {
    (void)hipEventSynchronize(ctx->upload_done);
    (void)hipEventDestroy(ctx->upload_done);
  }
  if (ctx->h_ptrs_pinned) (void)hipHostFree(ctx->h_ptrs_pinned);
  for (hipEvent_t ev : ctx->prof_events) (void)hipEventDestroy(ev);
  delete ctx;
}

const char* muon_status_string(int status) {
  switch (status) {
    case MUON_OK: return "ok";
    case MUON_E_INVALID_ARG: return "invalid argument";
    case MUON_E_UNSUPPORTED_DTYPE: return "unsupported dtype";
    case MUON_E_SHAPE_MISMATCH: return "parameter list does not match the one given at init";
    case MUON_E_WORKSPACE_TOO_SMALL: return "workspace too small";
    case MUON_E_HIP: return "HIP runtime error";
    case MUON_E_NOT_RESIDENT: return "matrix temporaries are not resident";
    case MUON_E_MISALIGNED: return "misaligned buffer";
    case MUON_E_NO_MEMORY: return "out of host memory";
    case MUON_E_STATIC_LIMIT: return "input exceeds the limits of muon_step_static";
    default: return "unknown status";
  }
}

int muon_last_hip_error(void) { return g_last_hip_error; }

}  // extern "C"
