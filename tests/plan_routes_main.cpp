// Which kernels the planner picks, on the host: built by tests/plan_routes.py with g++ together with
// paper_2502_16982_amd/csrc/muon_plan.cpp.  Arguments: ns dtype code, compute units, then rows and columns of every matrix.
// Output: a line "fold" per chunk with 1 where the first Gram launch adds up the norm.  Chunks without matrices of the Gram route: a
// line per product and level: chunk, product, level, entries of the table, form (whole, quarters, ring4, waves, ring128), last entries that
// run in quarters behind it.  Chunks with them: "pair", chunk, product of the matrices iterated as Eq. 2 is written (none, gram, sym,
// apply), of the others, entries of the fine launch, its form; "coarse", chunk, group, entries of the symmetric and of the apply product;
// "lone", chunk, entries, form alone, form with an apply product; "shared", chunk, entries; "joint", chunk, entries of both apply products,
// strips among them; "beside", chunk, group, product.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "../paper_2502_16982_amd/csrc/muon_plan.h"

using namespace muon;

static const char* form(bool quarters, int few) {
  return !quarters ? (few == 3 ? "ring128" : "whole") : few == 2 ? "waves" : few == 1 ? "ring4" : "quarters";
}

static void paired(size_t c, const Chunk& ch) {
  const char* const name[4] = {"none", "gram", "sym", "apply"};
  auto fine = [&](int group, int p) {
    const TileSet& t = ch.groups[group].fine;
    return p == kPairNone ? 0 : p == kPairGram ? t.n_sym : p == kPairSym ? t.n_poly : t.n_apply;
  };
  for (int i = 0; i < 4; ++i)
    for (int j = 0; j < 4; ++j)
      if (fine(0, i) + fine(1, j) > 0)
        std::printf("pair %zu %s %s %d %s\n", c, name[i], name[j], fine(0, i) + fine(1, j), form(ch.pair[i][j].quarters, ch.pair[i][j].few));
  for (int i = 0; i < 2; ++i) std::printf("coarse %zu %d %d %d\n", c, i, ch.groups[i].coarse.n_sym, ch.groups[i].coarse.n_apply);
  const Group& g = ch.groups[1];
  if (g.n_lone > 0)
    std::printf("lone %zu %d %s %s\n", c, g.n_lone, form(g.lone_form[0].quarters, g.lone_form[0].few), form(g.lone_form[1].quarters, g.lone_form[1].few));
  if (ch.n_shared_app > 0) std::printf("joint %zu %d %d\n", c, ch.n_shared_app, ch.shared_app_strips ? 1 : 0);
  if (ch.n_shared_sym > 0) std::printf("shared %zu %d\n", c, ch.n_shared_sym);
  for (int i = 0; i < 2; ++i)
    for (int p = 1; p < 4; ++p)
      if (ch.beside[i][p]) std::printf("beside %zu %d %s\n", c, i, name[p]);
}

int main(int argc, char** argv) {
  std::vector<muon_param> p;
  for (int i = 3; i + 1 < argc; i += 2) {
    muon_param q{};
    q.rows = std::atoll(argv[i]);
    q.cols = std::atoll(argv[i + 1]);
    q.w_dtype = q.g_dtype = MUON_BF16;
    p.push_back(q);
  }
  const int ns = std::atoi(argv[1]);
  Plan plan;
  plan.coarse_blocks = std::atoi(argv[2]);
  size_t bytes = 0;
  if (plan_workspace_bytes(p.data(), (int32_t)p.size(), ns, 0, &bytes) != MUON_OK) return 1;
  if (plan_build(plan, p.data(), (int32_t)p.size(), ns, uintptr_t{1} << 40, bytes) != MUON_OK) return 2;
  for (size_t c = 0; c < plan.chunks.size(); ++c) {
    std::printf("fold %d\n", plan.chunks[c].fold_norm ? 1 : 0);
    if (plan.chunks[c].paired) {
      paired(c, plan.chunks[c]);
      continue;
    }
    for (const Group& g : plan.chunks[c].groups)
      for (int level = 0; level < 2; ++level) {
        const TileSet& t = level ? g.coarse : g.fine;
        const int count[3] = {t.n_sym, t.n_poly, t.n_apply}, few[3] = {t.few_sym, t.few_poly, t.few_apply};
        const int tail[3] = {t.tail_sym, t.tail_poly, t.tail_apply};
        const bool quarters[3] = {t.quarter_sym, t.quarter_poly, t.quarter_apply};
        const char* const product[3] = {"gram", "poly", "apply"};
        for (int q = 0; q < 3; ++q)
          std::printf("%zu %s %d %d %s %d\n", c, product[q], level, count[q], form(quarters[q], few[q]), tail[q]);
      }
  }
  return 0;
}
