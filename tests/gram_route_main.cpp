// Tables of the Gram route, walked on the host under sanitizers: built by tests/test_gram_route.py with g++ together with
// paper_2502_16982_amd/csrc/muon_plan.cpp.
#include <cstdio>
#include <cstdlib>
#include <map>
#include <set>
#include <tuple>
#include <vector>

#include "../paper_2502_16982_amd/csrc/muon_plan.h"

using namespace muon;
static int failures = 0, beside = 0, joint = 0;
#define CHECK(c) do { if (!(c)) { if (failures++ < 20) std::printf("line %d: %s\n", __LINE__, #c); } } while (0)

typedef std::tuple<int, int, int, int> Key;      // problem, row, column, shape
static std::multiset<Key> keys(const GemmTile* t, int n, int second) {       // second: -1 any, 0 or 1 by the flag
  std::multiset<Key> out;
  for (int i = 0; i < n; ++i)
    if (second < 0 || ((t[i].flags & kTileSecond) != 0) == (second == 1)) out.insert(Key(t[i].prob, t[i].r0, t[i].c0, t[i].shape));
  return out;
}

static void walk(const std::vector<muon_param>& p, size_t cap) {
  size_t bytes = 0;
  CHECK(plan_workspace_bytes(p.data(), (int32_t)p.size(), MUON_BF16, cap, &bytes) == MUON_OK);
  Plan plan;
  const uintptr_t base = uintptr_t{1} << 40;
  const int st = plan_build(plan, p.data(), (int32_t)p.size(), MUON_BF16, base, bytes);
  CHECK(st == MUON_OK);
  if (st != MUON_OK) return;
  unsigned char* const img = plan.image.data();
  const MatDesc* mats = reinterpret_cast<const MatDesc*>(img + plan.off_mats);
  for (const Chunk& ch : plan.chunks) {
    bool any = false;
    for (int i = ch.first; i < ch.first + ch.count; ++i) {
      any = any || plan.mats[i].gram;
      CHECK(mats[i].gram_route == (int)plan.mats[i].gram);
    }
    CHECK(ch.paired == any && ch.groups.size() == (any ? 2u : 1u));
    if (!any) continue;
    for (int r = 0; r < 2; ++r) {
      const Group& g = ch.groups[r];
      CHECK(g.gram == (r == 1) || g.n_prob == 0);
      for (int i : g.members) CHECK((int)plan.mats[i].gram == r);
    }
    const Group& g = ch.groups[1];
    CHECK(g.prob_ops + sizeof(GemmProblem) * (size_t)g.n_prob * kGramOps <= plan.image.size());
    const GemmProblem* ops = reinterpret_cast<const GemmProblem*>(img + g.prob_ops);
    for (int k = 0; k < g.n_prob; ++k) {
      const MatPlan& q = plan.mats[g.members[k]];
      const MatDesc& d = mats[g.members[k]];
      const size_t ab = 2 * (size_t)q.mp * q.mp, xb = 2 * (size_t)q.mp * q.np;
      CHECK(ab <= xb);
      auto in = [](const void* v, size_t n, const void* from, size_t room) {
        const uintptr_t a = (uintptr_t)v, f = (uintptr_t)from;
        return a >= f && a + n <= f + room;
      };
      for (int par = 0; par < 2; ++par) {
        const void* const other = par ? d.X : d.Xt[0];
        const void* const x = par ? d.Xt[0] : d.X;
        auto small = [&](const void* v) { return in(v, ab, d.Ag, ab) || in(v, ab, d.Bp, ab) || in(v, ab, other, xb); };
        for (int o = 0; o < kGramParityOps; ++o) {
          const GemmProblem& s = ops[(par * kGramParityOps + o) * g.n_prob + k];
          CHECK(small(s.L) && small(s.R) && small(s.C) && (!s.Et || small(s.Et)) && s.Ct == nullptr);
          CHECK(s.C != s.L && s.C != s.R && s.C != s.Et);                  // nothing is written that the same launch reads
          CHECK(s.K == q.mp && s.ldl == q.mp && s.ldr == q.mp && s.ldc == q.mp && s.diag_add == 0);
          CHECK(s.symmetric == (s.L == s.R ? 1 : kMirrored));
        }
        for (int last = 0; last < 2; ++last) {
          const GemmProblem& s = ops[(kGramApply + par * 2 + last) * g.n_prob + k];
          CHECK(s.L == x && s.R == d.Ag && s.Et == nullptr && s.K == q.mp && s.ldl == q.np);
          CHECK(last && q.transposed ? s.C == d.Xt[1] && !s.Ct : s.Ct == other && !s.C);
        }
      }
    }
    for (int i = 0; i < 2; ++i)
      for (int j = 0; j < 2 && ch.n_shared_sym > 0; ++j) {
        CHECK(ch.shared_sym[i][j] + sizeof(GemmTile) * (size_t)ch.n_shared_sym <= plan.image.size());
        const GemmTile* t = reinterpret_cast<const GemmTile*>(img + ch.shared_sym[i][j]);
        for (int r = 0; r < 2; ++r) {
          const TileSet& c = ch.groups[r].coarse;
          CHECK(keys(t, ch.n_shared_sym, r) == keys(reinterpret_cast<const GemmTile*>(img + c.sym), c.n_sym, -1));
        }
      }
    if (ch.n_shared_app > 0) {           // a group's own coarse tiles, or coarse tiles over all of its outputs
      CHECK(ch.shared_app + sizeof(GemmTile) * (size_t)ch.n_shared_app <= plan.image.size());
      const GemmTile* t = reinterpret_cast<const GemmTile*>(img + ch.shared_app);
      for (int r = 0; r < 2; ++r) {
        const Group& h = ch.groups[r];
        const std::multiset<Key> own = keys(t, ch.n_shared_app, r);
        if (h.coarse.n_apply > 0) {
          CHECK(own == keys(reinterpret_cast<const GemmTile*>(img + h.coarse.apply), h.coarse.n_apply, -1));
          continue;
        }
        std::vector<std::set<std::pair<int, int>>> seen(h.members.size());
        for (const Key& k : own) {
          const int rows = kShapeRows[std::get<3>(k)] / kTileUnit, cols = kShapeCols[std::get<3>(k)] / kTileUnit;
          CHECK(std::get<0>(k) >= 0 && std::get<0>(k) < h.n_prob);
          CHECK(std::get<3>(k) == (int)kShape256 || (std::get<3>(k) == (int)kShape512x128 && ch.shared_app_strips));
          for (int a = 0; a < rows; ++a)
            for (int b = 0; b < cols; ++b) seen[std::get<0>(k)].insert({std::get<1>(k) + a, std::get<2>(k) + b});
        }
        for (size_t k = 0; k < seen.size(); ++k) {
          const MatPlan& q = plan.mats[h.members[k]];
          CHECK(seen[k].size() == (size_t)(q.np / kTileUnit) * (q.mp / kTileUnit) && seen[k].rbegin()->first == q.np / kTileUnit - 1);
          int last = 0;
          for (const auto& at : seen[k]) last = std::max(last, at.second);
          CHECK(last == q.mp / kTileUnit - 1);
        }
        joint += 1;
      }
    }
    for (int i = 0; i < 2; ++i)
      for (int p : {kPairGram, kPairSym, kPairApply}) {        // blocks of a ring beside coarse tiles: all of the product in them, K of four slabs
        if (!ch.beside[i][p]) continue;
        const Group& h = ch.groups[i];
        const bool lone = p == kPairSym && h.n_lone > 0;
        CHECK(lone || (p == kPairApply ? h.coarse.n_apply == 0 && h.fine.n_apply > 0 : h.coarse.n_sym == 0 && h.fine.n_sym > 0));
        CHECK(ch.groups[i ^ 1].coarse.n_apply > 0);
        for (int k : h.members) CHECK(plan.mats[k].mp >= 256);
        ++beside;
      }
    if (g.n_lone > 0) {
      CHECK(g.lone + sizeof(GemmTile) * (size_t)g.n_lone <= plan.image.size());
      const GemmTile* t = reinterpret_cast<const GemmTile*>(img + g.lone);
      std::multiset<Key> want;
      for (int k = 0; k < g.n_prob; ++k) {
        const int n = plan.mats[g.members[k]].mp / 128;
        for (int a = 0; a < n; ++a)
          for (int b = a; b < n; ++b) want.insert(Key(k, 2 * a, 2 * b, (int)kShape128));
      }
      CHECK(keys(t, g.n_lone, -1) == want);
    }
  }
}

static muon_param mat(int64_t a, int64_t b) {
  muon_param q{};
  q.rows = a;
  q.cols = b;
  q.w_dtype = q.g_dtype = MUON_BF16;
  return q;
}

int main() {
  // the line itself
  struct { int64_t a, b; bool gram; } const edge[] = {
      {256, 1 << 17, false}, {257, 3072, true}, {384, 2944, false}, {2945, 384, true}, {512, 3968, false}, {512, 4096, true}, {640, 2432, false},
      {2433, 640, true}, {1024, 3968, false}, {1024, 3969, true}, {1152, 4480, false}, {1153, 3328, true}, {1280, 3200, false}, {1280, 3328, true}, {2432, 6272, false},
      {2433, 5120, true}, {2560, 5120, true}, {2561, 5248, false}, {4096, 11008, true}, {2048, 2048, false}};
  for (const auto& e : edge) {
    Plan plan;
    const muon_param p = mat(e.a, e.b);
    for (int ns : {MUON_BF16, MUON_BF16X2, MUON_BF16X3, MUON_F32}) {
      size_t bytes = 0;
      CHECK(plan_workspace_bytes(&p, 1, ns, 0, &bytes) == MUON_OK);
      CHECK(plan_build(plan, &p, 1, ns, uintptr_t{1} << 40, bytes) == MUON_OK);
      if (plan.mats[0].gram != (e.gram && ns == MUON_BF16)) std::printf("%d x %d, arithmetic %d\n", (int)e.a, (int)e.b, ns), ++failures;
    }
  }
  std::srand(7);
  auto rnd = [](int lo, int hi) { return lo + std::rand() % (hi - lo + 1); };
  for (int it = 0; it < 60; ++it) {
    std::vector<muon_param> p;
    const int kinds = rnd(1, 4);
    for (int k = 0; k < kinds; ++k) {
      const int64_t m = rnd(300, 1500), n = k % 2 ? rnd(16, 1600) : m * rnd(2, 9) + rnd(0, 200);
      for (int c = rnd(1, it % 3 ? 4 : 30); c > 0; --c) p.push_back(c % 2 ? mat(m, n) : mat(n, m));
    }
    walk(p, 0);
    walk(p, 1);                       // one matrix at a time
    walk(p, (size_t)64 << 20);
  }
  // groups: one iteration as it is written, twos, and one where one is left
  for (int n = kGramMinSteps; n <= 40; ++n) {
    int it = 0, count = 0;
    for (; it < n; ++count) {
      const int k = gram_group(it, n);
      CHECK(k == (it == 0 || it == n - 1 ? 1 : 2));
      it += k;
    }
    CHECK(it == n && count == gram_groups(n));
  }
  // coefficients: the paper's up to ten iterations; large ones, ones that only grow on the way, and ones under which X shrinks
  double gain = 0.0;
  std::vector<double> c;
  for (int i = 0; i < 40; ++i) for (double v : {3.4445, -4.7750, 2.0315}) c.push_back(v);
  for (int n = kGramMinSteps; n <= 40; ++n) CHECK(gram_coefficients_fit(c.data(), n, &gain) == (n <= 10));
  std::vector<double> far = c;
  far[0] = 100.0; far[1] = far[2] = 0.0;
  CHECK(!gram_coefficients_fit(far.data(), 5, &gain));
  far = c;
  for (int i = 6; i < 15; ++i) far[i] = i % 3 ? 0.0 : 6.0;
  CHECK(!gram_coefficients_fit(far.data(), 5, &gain) && !gram_coefficients_fit(far.data(), 4, &gain));
  CHECK(gram_coefficients_fit(c.data(), 5, &gain) && gain >= 484.9 && gain <= 1.25 * 485.0);           // 3.4445^5
  far = c;
  far[0] = 0.01; far[3] = 100.0; far[1] = far[2] = far[4] = far[5] = 0.0;
  CHECK(!gram_coefficients_fit(far.data(), 5, &gain));                                                 // X shrinks
  const double textbook[12] = {1.875, -1.25, 0.375, 1.875, -1.25, 0.375, 1.5, -0.5, 0.0, 1.0, 0.0, 0.0};
  CHECK(gram_coefficients_fit(textbook, 4, &gain));
  const std::vector<muon_param> few = {mat(3000, 3000), mat(1024, 4096)}, full = {mat(2048, 2048), mat(2048, 2048), mat(2048, 2048), mat(2048, 2048),
                                                                                   mat(2048, 2048), mat(2048, 2048), mat(2048, 2048), mat(2048, 2048), mat(1024, 4096)};
  CHECK(joint > 0);
  beside = joint = 0;
  walk(few, 0);
  CHECK(beside == 3 && joint == 1);
  walk(full, 0);                      // 512 apply tiles: no compute unit is idle
  CHECK(beside == 3 && joint == 1);
  std::printf(failures ? "failed\n" : "gram route ok\n");
  return failures ? 1 : 0;
}
