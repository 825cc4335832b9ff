// Which kernels the planner picks, on the host: built by tests/plan_routes.py with g++ together with
// paper_2502_16982_amd/csrc/muon_plan.cpp.  Arguments: ns dtype code, compute units, then rows and columns of every matrix.
// Output, a line per chunk, product and level: chunk, product, level, entries of the table, form (whole, quarters, ring4, waves);
// and a line "fold" with 1 where the first Gram launch adds up the norm.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "../paper_2502_16982_amd/csrc/muon_plan.h"

int main(int argc, char** argv) {
  using namespace muon;
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
    for (const Group& g : plan.chunks[c].groups)
      for (int level = 0; level < 2; ++level) {
        const TileSet& t = level ? g.coarse : g.fine;
        const int count[3] = {t.n_sym, t.n_poly, t.n_apply}, few[3] = {t.few_sym, t.few_poly, t.few_apply};
        const bool quarters[3] = {t.quarter_sym, t.quarter_poly, t.quarter_apply};
        const char* const product[3] = {"gram", "poly", "apply"};
        for (int q = 0; q < 3; ++q)
          std::printf("%zu %s %d %d %s\n", c, product[q], level, count[q],
                      !quarters[q] ? "whole" : few[q] == 2 ? "waves" : few[q] == 1 ? "ring4" : "quarters");
      }
  }
  return 0;
}
