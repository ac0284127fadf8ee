// Test harness (host only): plans the resident CG of problems read from a binary file
// and prints the plan as text.  Input: int32 n_probs, n_blocks, target slots, then per
// problem int64 first oct and octs, then int64 rows and int32 nbr[rows][6], and of a
// system with couplings between levels int32 cnb[rows][6] and child[8 rows].  Output:
// the shares (slot0 n_slots unit0 n_units prob part0 group), unit_of, partner, task0, task,
// the largest share and its units, places; with couplings the shares' coarse units,
// coarse, couplings; last the peers and the length of the near numbering.
#include <cstdio>
#include <vector>

#include "resident_plan.h"

int main(int argc, char** argv) {
  if (argc != 2) return 2;
  FILE* f = std::fopen(argv[1], "rb");
  if (!f) return 2;
  int32_t head[3];
  if (std::fread(head, 4, 3, f) != 3) return 2;
  std::vector<amrfld::ResProblem> probs(head[0]);
  std::vector<int> group;
  for (auto& p : probs) {
    int64_t v[2];
    if (std::fread(v, 8, 2, f) != 2) return 2;
    p.oct0 = v[0];
    p.n_oct = v[1];
    p.id = int(&p - probs.data());
    group.push_back(amrfld::res_group(p.n_oct, head[1], head[2], head[2]));
  }
  int64_t rows = 0;
  if (std::fread(&rows, 8, 1, f) != 1) return 2;
  std::vector<int32_t> nbr(6 * rows);
  if (std::fread(nbr.data(), 4, nbr.size(), f) != nbr.size()) return 2;
  std::vector<int32_t> cnb(6 * rows), child(8 * rows);
  const bool coupled = std::fread(cnb.data(), 4, cnb.size(), f) == cnb.size() &&
                       std::fread(child.data(), 4, child.size(), f) == child.size();
  std::fclose(f);
  const amrfld::ResPlanHost h =
      amrfld::build_res_plan(probs, group, head[1], nbr.data(), rows, coupled ? cnb.data() : nullptr,
                             coupled ? child.data() : nullptr);
  auto line = [](const std::vector<int32_t>& v) {
    for (size_t i = 0; i < v.size(); ++i) std::printf(i ? " %d" : "%d", v[i]);
    std::printf("\n");
  };
  std::vector<int32_t> parts;
  for (const auto& p : h.parts)
    for (int v : {p.slot0, p.n_slots, p.unit0, p.n_units, p.prob, p.part0, p.group}) parts.push_back(v);
  line(parts);
  line(h.unit_of);
  line(h.partner);
  line(h.task0);
  line(h.task);
  std::printf("%d %d\n", h.max_slots, h.max_units);
  line(std::vector<int32_t>(h.places.begin(), h.places.end()));
  if (coupled) {
    std::vector<int32_t> n;
    for (const auto& p : h.parts) n.push_back(p.n_coarse);
    line(n);
    line(h.coarse);
    line(std::vector<int32_t>(h.couplings.begin(), h.couplings.end()));
  }
  std::vector<int32_t> peers(h.peers);
  peers.push_back(h.n_near);
  line(peers);
  return 0;
}
