// Test harness (host only): the plan of boxes of m^3 octs, one after another, made by one
// thread and by several; prints "same" where every table is.  Arguments: threads, n_blocks,
// target slots, then m of each box.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "resident_plan.h"

using namespace amrfld;

template <class A, class B>
static bool equal(const A& a, const B& b) {
  return a.size() == b.size() && std::equal(a.begin(), a.end(), b.begin());
}

int main(int argc, char** argv) {
  if (argc < 5) return 2;
  const int threads = std::atoi(argv[1]), n_blocks = std::atoi(argv[2]), target = std::atoi(argv[3]);
  std::vector<ResProblem> probs;
  std::vector<int> group;
  std::vector<int32_t> nbr;
  for (int k = 4; k < argc; ++k) {
    const int m = std::atoi(argv[k]);
    ResProblem p;
    p.oct0 = int64_t(nbr.size() / 6);
    p.n_oct = int64_t(m) * m * m;
    p.id = k - 4;
    for (int z = 0; z < m; ++z)
      for (int y = 0; y < m; ++y)
        for (int x = 0; x < m; ++x) {
          const int32_t o = int32_t(p.oct0 + (int64_t(z) * m + y) * m + x), mm = m * m;
          for (int32_t v : {x > 0 ? o - 1 : -1, x + 1 < m ? o + 1 : -1, y > 0 ? o - m : -1, y + 1 < m ? o + m : -1,
                            z > 0 ? o - mm : -1, z + 1 < m ? o + mm : -1})
            nbr.push_back(v);
        }
    nbr.insert(nbr.end(), 18, -1);  // rows that no problem uses
    group.push_back(res_group(p.n_oct, n_blocks, target, target));
    probs.push_back(p);
  }
  const int64_t rows = int64_t(nbr.size() / 6);
  const ResPlanHost a = build_res_plan(probs, group, n_blocks, nbr.data(), rows, nullptr, nullptr, true, 1);
  const ResPlanHost b = build_res_plan(probs, group, n_blocks, nbr.data(), rows, nullptr, nullptr, true, threads);
  bool same = equal(a.unit_of, b.unit_of) && equal(a.partner, b.partner) && equal(a.peers, b.peers) &&
              equal(a.task0, b.task0) && equal(a.task, b.task) && a.n_near == b.n_near && a.max_units == b.max_units &&
              a.max_slots == b.max_slots && a.parts.size() == b.parts.size() &&
              std::memcmp(a.parts.data(), b.parts.data(), a.parts.size() * sizeof(ResPart)) == 0;
  for (const ResPart& p : a.parts)
    same = same && std::equal(a.places.begin() + p.slot0, a.places.begin() + p.slot0 + p.n_slots,
                              b.places.begin() + p.slot0);
  std::printf(same ? "same %zu\n" : "other %zu\n", a.partner.size());
  return 0;
}
