// Pulled sequences of the best responses on a plan made up of two pieces: a
// deep one with three external parents, whose rows start at `first`, and one
// above it that pulls their values over two wavefronts.
#include "pmx_internal.hpp"

using namespace pmx;

extern "C" int check_rm_pull_seqs(int first) {
  RmPlan P;
  P.n_slot = 3;
  RmTask deep{}, top{};
  deep.n_rows = 4;
  deep.n_ext = 3;
  P.rows = {first, first + 7, first + 8, first + 20, 0, 1, 2};
  P.ext_slot = {2, 0, 1};
  P.ext_seq = {0, 1, 2};
  top.rows_off = 4;
  top.n_rows = 3;
  P.pulls.assign(kRmGroups, 0);
  P.pulls[0] = 2;
  P.pulls[1] = 1;
  P.pulls.insert(P.pulls.end(), {40 | 2 << 8, 44 | 1 << 8, 41 | 0 << 8});
  top.n_pull = (int)P.pulls.size();
  P.tasks = {deep, top};
  const std::vector<int32_t> s = rm_pull_seqs(P);
  if (s.size() != P.pulls.size()) return 1;
  for (int w = 0; w < kRmGroups; ++w)
    if (s[w] != 0) return 2;
  if (s[kRmGroups] != first || s[kRmGroups + 1] != first + 8 || s[kRmGroups + 2] != first + 7) return 3;
  return 0;
}
