// Shares and halo faces of the resident CG (host).
#include "resident_plan.h"

#include <algorithm>

namespace amrfld {

int res_group(int64_t n_oct, int max_blocks, int max_slots, int target_slots) {
  if (8 * n_oct <= max_slots) return 1;
  const int64_t want = (8 * n_oct + target_slots - 1) / target_slots;
  int64_t g = std::max<int64_t>(1, std::min<int64_t>({want, n_oct, int64_t(max_blocks)}));
  if (g > 8) g = std::min<int64_t>((g + 7) / 8 * 8, max_blocks);  // as many blocks on every XCD
  return int(std::min<int64_t>(g, n_oct));
}

int res_blocks(int g, int n_cu) {
  const int per = std::max(1, n_cu / 8);  // compute units of an XCD
  const int n_xcd = (g + per - 1) / per;
  // (never fewer than shares: units that are no multiple of 8 leave an XCD over)
  return g == 1 ? 1 : std::max(g, std::min(n_cu, 8 * ((g + n_xcd - 1) / n_xcd)));
}

double res_cost(int n_slots, int group) {
  return 0.6 + 0.0005 * n_slots + (group > 1 ? 2.5 + 0.012 * group : 0.0);
}

ResPlanHost build_res_plan(const std::vector<ResProblem>& probs, const std::vector<int>& group, int n_blocks,
                           const int32_t* nbr, int64_t n_oct_table, const int32_t* cnb, const int32_t* child) {
  ResPlanHost h;
  std::vector<int32_t> part_of(n_oct_table, -1);
  for (size_t q = 0; q < probs.size(); ++q) {
    const int64_t m = probs[q].n_oct;
    const int g = group[q], p0 = int(h.parts.size());
    // even shares; with couplings between levels even in slots and, counted twice, in faces
    // towards finer cells (a share of 1400 slots beside a refined region has up to as many,
    // whose halo would not fit LDS and whose exchange every other share waits for)
    std::vector<int64_t> first(g + 1);
    for (int r = 0; r <= g; ++r) first[r] = probs[q].oct0 + m * r / g;
    if (cnb) {
      std::vector<int64_t> w(m, 8);
      for (int64_t o = 0; o < n_oct_table; ++o)
        for (int d = 0; d < 6; ++d)
          if (nbr[6 * o + d] < 0 && cnb[6 * o + d] >= 0) w[cnb[6 * o + d] / 8 - probs[q].oct0] += 2;
      int64_t total = 0, sum = 0;
      for (int64_t x : w) total += x;
      for (int64_t o = 0, r = 1; o < m && r < g; ++o) {
        sum += w[o];
        // (at least one oct to every share, before and after)
        if ((sum * g >= total * r && o + 1 >= r) || m - (o + 1) <= g - r) first[r++] = probs[q].oct0 + o + 1;
      }
    }
    for (int r = 0; r < g; ++r) {
      const int64_t o0 = first[r], o1 = first[r + 1];
      ResPart p{};
      p.slot0 = int(8 * o0);
      p.n_slots = int(8 * (o1 - o0));
      p.prob = probs[q].id;
      p.part0 = p0;
      p.group = g;
      for (int64_t o = o0; o < o1; ++o) part_of[o] = int32_t(h.parts.size());
      h.max_slots = std::max(h.max_slots, p.n_slots);
      h.parts.push_back(p);
    }
  }
  h.unit_of.assign(6 * n_oct_table, -1);
  int32_t n_units = 0;
  for (ResPart& p : h.parts) {
    p.unit0 = n_units;
    const int32_t me = part_of[p.slot0 / 8];
    for (int64_t o = p.slot0 / 8; o < (int64_t(p.slot0) + p.n_slots) / 8; ++o)
      for (int d = 0; d < 6; ++d) {
        const int32_t nb = nbr[6 * o + d];
        if (nb >= 0 ? part_of[nb] != me : cnb && cnb[6 * o + d] >= 0) h.unit_of[6 * o + d] = n_units++;
      }
    if (cnb) {
      // the leaves' faces towards finer cells, slot by slot
      const int32_t first = n_units;
      h.couplings.resize(4 * n_oct_table, 0u);
      for (int64_t i = p.slot0; i < int64_t(p.slot0) + p.n_slots; ++i) {
        if (child[i] != -1) continue;
        const int pos = int(i & 7);
        for (int d = 0; d < 6; ++d) {
          const int a = d >> 1, bit = 1 << a;
          const int32_t nb = nbr[6 * (i >> 3) + d];
          const int64_t j = ((pos >> a) & 1) != (d & 1) ? i ^ bit : nb >= 0 ? (int64_t(nb) << 3) | (pos ^ bit) : -1;
          if (j < 0 || child[j] < 0) continue;
          uint32_t& c = h.couplings[i >> 1];
          if (c == 0) c = uint32_t(n_units - first);
          c += i & 1 ? 1u << 24 : 1u << 16;
          h.coarse.resize(2 * size_t(n_units) + 2, 0);
          h.coarse[2 * size_t(n_units)] = int32_t(i - p.slot0);
          h.coarse[2 * size_t(n_units) + 1] = 8 * child[j] + (d ^ 1);
          ++n_units;
        }
      }
      p.n_coarse = n_units - first;
    }
    p.n_units = n_units - p.unit0;
    h.max_units = std::max(h.max_units, p.n_units);
  }
  h.partner.assign(n_units, -1);
  for (const ResPart& p : h.parts)
    for (int64_t o = p.slot0 / 8; o < (int64_t(p.slot0) + p.n_slots) / 8; ++o)
      for (int d = 0; d < 6; ++d) {
        const int32_t u = h.unit_of[6 * o + d];
        if (u >= 0 && nbr[6 * o + d] >= 0) h.partner[u] = h.unit_of[6 * int64_t(nbr[6 * o + d]) + (d ^ 1)];
      }
  if (cnb) h.coarse.resize(2 * size_t(n_units), 0);
  for (const ResPart& p : h.parts)
    for (int32_t u = p.unit0 + p.n_units - p.n_coarse; u < p.unit0 + p.n_units; ++u) {
      const int32_t f = h.unit_of[6 * int64_t(h.coarse[2 * u + 1] >> 3) + (h.coarse[2 * u + 1] & 7)];
      h.partner[u] = f;
      h.partner[f] = u;
    }
  std::vector<int32_t> share_of(n_units);
  for (size_t k = 0; k < h.parts.size(); ++k)
    std::fill_n(share_of.begin() + h.parts[k].unit0, h.parts[k].n_units, int32_t(k));
  h.n_near = ResPlanHost::near_base(n_units, int32_t(h.parts.size()));
  h.peers.resize(2 * size_t(n_units));
  for (int32_t u = 0; u < n_units; ++u) {
    const int32_t k = share_of[h.partner[u]];
    const ResPart& p = h.parts[k];
    h.peers[2 * size_t(u)] = ResPlanHost::near_base(p.unit0, k) + (h.partner[u] - p.unit0);
    h.peers[2 * size_t(u) + 1] = k - p.part0;
  }
  h.places.assign(8 * n_oct_table, 0);
  for (const ResPart& p : h.parts)
    for (int64_t o = p.slot0 / 8; o < (int64_t(p.slot0) + p.n_slots) / 8; ++o)
      for (int k = 0; k < 4; ++k) {  // pair k of the oct: y = k & 1, z = k >> 1
        const unsigned own = unsigned(8 * o + 2 * k - p.slot0);
        auto place = [&](int d, unsigned self, unsigned inside, unsigned cell) -> unsigned {
          const int32_t nb = nbr[6 * o + d], u = h.unit_of[6 * o + d];
          if (u >= 0) return kResHalo | unsigned(4 * (u - p.unit0)) + cell;
          return nb < 0 ? self : unsigned(8 * int64_t(nb) - p.slot0) + inside;
        };
        const int y = k & 1, z = k >> 1;
        const unsigned x0 = place(0, own, unsigned(2 * k + 1), unsigned(k)), x1 = place(1, own + 1, unsigned(2 * k), unsigned(k));
        const unsigned py = place(2 + y, own, unsigned(2 * (k ^ 1)), unsigned(2 * z));
        const unsigned pz = place(4 + z, own, unsigned(2 * (k ^ 2)), unsigned(2 * y));
        h.places[8 * o + 2 * k] = x0 | (x1 << 16);
        h.places[8 * o + 2 * k + 1] = py | (pz << 16);
      }
  // Blocks: each problem goes to the `group` least loaded blocks.  Every block works on
  // its shares in the order of the problems, so the first unfinished problem always has
  // all its blocks on it: no block waits for one that waits for it.
  // Blocks are dealt to the XCDs round-robin, and shares on the same XCD exchange through
  // its L2: neighbouring shares go to the same XCD, as far as the loads allow.
  struct Block {
    double time;
    int id;
  };
  auto by_xcd = [](const Block& a, const Block& b) {
    return std::make_pair(a.id % 8, a.id) < std::make_pair(b.id % 8, b.id);
  };
  auto by_load = [&](const Block& a, const Block& b) { return a.time != b.time ? a.time < b.time : by_xcd(a, b); };
  // The order in which a problem's shares are dealt to its blocks: theirs, which puts
  // neighbours on a level on one XCD (80 to 90 % of the units of a refined level), and
  // with couplings between levels the one that grows clusters of an XCD's size by the
  // units shared (in order a share of the finest level has 20 % of its units there).
  std::vector<int32_t> deal(h.parts.size());
  for (size_t k = 0; k < deal.size(); ++k) deal[k] = int32_t(k);
  if (cnb) {
    const int g = int(deal.size()), size = (g + 7) / 8;
    std::vector<std::vector<std::pair<int32_t, int32_t>>> near(g);
    std::vector<int32_t> count(g, 0);
    for (int k = 0; k < g; ++k) {
      const ResPart& p = h.parts[k];
      for (int32_t u = p.unit0; u < p.unit0 + p.n_units; ++u) ++count[share_of[h.partner[u]]];
      for (int j = 0; j < g; ++j)
        if (count[j]) near[k].push_back({j, count[j]}), count[j] = 0;
    }
    std::vector<char> used(g, 0);
    std::vector<int64_t> gain(g, 0);
    for (int n = 0; n < g; ++n) {
      if (n % size == 0) std::fill(gain.begin(), gain.end(), 0);
      int best = -1;
      for (int k = 0; k < g; ++k)
        if (!used[k] && (best < 0 || gain[k] > gain[best])) best = k;
      used[best] = 1;
      deal[n] = best;
      for (const auto& e : near[best]) gain[e.first] += e.second;
    }
  }
  std::vector<std::vector<int32_t>> list(n_blocks);
  std::vector<Block> load(n_blocks);
  for (int b = 0; b < n_blocks; ++b) load[b] = {0.0, b};
  for (size_t q = 0, at = 0; q < probs.size(); at += size_t(group[q]), ++q) {
    const int g = group[q];
    std::partial_sort(load.begin(), load.begin() + g, load.end(), by_load);
    std::sort(load.begin(), load.begin() + g, by_xcd);
    double end = 0.0;  // the problem begins when the last of its blocks is free
    for (int r = 0; r < g; ++r) end = std::max(end, load[r].time);
    end += res_cost(h.parts[at].n_slots, g);
    for (int r = 0; r < g; ++r) {
      list[load[r].id].push_back(deal[at + r]);
      load[r].time = end;
    }
  }
  h.task0.assign(1, 0);
  for (int b = 0; b < n_blocks; ++b) {
    h.task.insert(h.task.end(), list[b].begin(), list[b].end());
    h.task0.push_back(int32_t(h.task.size()));
  }
  return h;
}

}  // namespace amrfld
