// Shares and halo faces of the resident CG (host).
#include "resident_plan.h"

#include <algorithm>
#include <atomic>
#include <condition_variable>
#include <mutex>
#include <system_error>
#include <thread>

namespace amrfld {

namespace {

// Threads that work on the shares of a plan, pass after pass, the calling one among them.
class Team {
 public:
  explicit Team(int threads) {
    more_.reserve(size_t(std::max(0, threads - 1)));
    try {
      while (int(more_.size()) < threads - 1) more_.emplace_back([this] { follow(); });
    } catch (const std::system_error&) {  // no more threads to be had: those there are will do
    }
  }
  ~Team() {
    {
      std::lock_guard<std::mutex> lk(mu_);
      pass_ = -1;
    }
    begin_.notify_all();
    for (std::thread& t : more_) t.join();
  }
  // f(k) for k = 0 .. n - 1.  f throws nothing and writes nothing that another call reads.
  template <class F>
  void each(int n, const F& f) {
    if (more_.empty()) {
      for (int k = 0; k < n; ++k) f(k);
      return;
    }
    next_ = 0;
    {
      std::lock_guard<std::mutex> lk(mu_);
      call_ = [](const void* g, int k) { (*static_cast<const F*>(g))(k); };
      f_ = &f;
      n_ = n;
      busy_ = int(more_.size());
      ++pass_;
    }
    begin_.notify_all();
    work();
    std::unique_lock<std::mutex> lk(mu_);
    end_.wait(lk, [this] { return busy_ == 0; });
  }

 private:
  void work() {
    for (int k = next_.fetch_add(1); k < n_; k = next_.fetch_add(1)) call_(f_, k);
  }
  void follow() {
    std::unique_lock<std::mutex> lk(mu_);
    for (int64_t seen = 0;;) {
      begin_.wait(lk, [&] { return pass_ != seen; });
      if (pass_ < 0) return;
      seen = pass_;
      lk.unlock();
      work();
      lk.lock();
      if (--busy_ == 0) end_.notify_one();
    }
  }
  std::vector<std::thread> more_;
  std::mutex mu_;
  std::condition_variable begin_, end_;
  std::atomic<int> next_{0};
  int64_t pass_ = 0;
  int n_ = 0, busy_ = 0;
  void (*call_)(const void*, int) = nullptr;
  const void* f_ = nullptr;
};

}  // namespace

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
                           const int32_t* nbr, int64_t n_oct_table, const int32_t* cnb, const int32_t* child,
                           bool faces, int threads) {
  ResPlanHost h;
  if (threads <= 0)
    threads = int(std::min<int64_t>({kResPlanThreads, int64_t(std::max(1u, std::thread::hardware_concurrency())),
                                     1 + n_oct_table / kResPlanThreadOcts}));
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
      h.max_slots = std::max(h.max_slots, p.n_slots);
      h.parts.push_back(p);
    }
  }
  const int n_parts = int(h.parts.size());
  Team team(std::min(threads, n_parts));
  auto oct0 = [&](const ResPart& p) { return int64_t(p.slot0) / 8; };
  auto oct1 = [&](const ResPart& p) { return (int64_t(p.slot0) + p.n_slots) / 8; };
  // f(slot, direction, finer oct) for the share's leaves' faces towards finer cells, slot by slot
  auto towards_finer = [&](const ResPart& p, auto f) {
    for (int64_t i = p.slot0; i < int64_t(p.slot0) + p.n_slots; ++i) {
      if (child[i] != -1) continue;
      const int pos = int(i & 7);
      for (int d = 0; d < 6; ++d) {
        const int a = d >> 1, bit = 1 << a;
        const int32_t nb = nbr[6 * (i >> 3) + d];
        const int64_t j = ((pos >> a) & 1) != (d & 1) ? i ^ bit : nb >= 0 ? (int64_t(nb) << 3) | (pos ^ bit) : -1;
        if (j >= 0 && child[j] >= 0) f(i, d, child[j]);
      }
    }
  };
  // the units counted, then numbered share by share
  ResArray<uint8_t> outer(n_oct_table);  // bit d: the oct's face d has a halo unit
  team.each(n_parts, [&](int k) {
    ResPart& p = h.parts[k];
    const int64_t o0 = oct0(p), o1 = oct1(p);
    int32_t n = 0;
    for (int64_t o = o0; o < o1; ++o) {
      unsigned m = 0;
      for (int d = 0; d < 6; ++d) {
        const int32_t nb = nbr[6 * o + d];
        m |= unsigned(nb >= 0 ? nb < o0 || nb >= o1 : cnb && cnb[6 * o + d] >= 0) << d;
      }
      outer[o] = uint8_t(m);
      n += __builtin_popcount(m);
    }
    if (cnb) towards_finer(p, [&](int64_t, int, int32_t) { ++p.n_coarse; });
    p.n_units = n + p.n_coarse;
  });
  int32_t n_units = 0;
  for (ResPart& p : h.parts) {
    p.unit0 = n_units;
    n_units += p.n_units;
    h.max_units = std::max(h.max_units, p.n_units);
  }
  ResArray<int32_t> unit0(n_oct_table);  // first unit of an oct
  auto unit_of = [&](int64_t face) {
    const int64_t o = face / 6;
    return unit0[o] + __builtin_popcount(outer[o] & ((1u << (face % 6)) - 1u));
  };
  std::vector<int32_t> share_of(n_units);
  h.places.resize(8 * n_oct_table);
  if (faces) h.unit_of.assign(6 * n_oct_table, -1);
  if (cnb) {
    h.couplings.resize(4 * n_oct_table, 0u);
    h.coarse.resize(2 * size_t(n_units), 0);
  }
  team.each(n_parts, [&](int k) {
    const ResPart& p = h.parts[k];
    std::fill_n(share_of.begin() + p.unit0, p.n_units, int32_t(k));
    int32_t next = p.unit0;
    for (int64_t o = oct0(p); o < oct1(p); ++o) {
      int32_t unit[6];
      unit0[o] = next;
      for (int d = 0; d < 6; ++d) {
        unit[d] = (outer[o] >> d) & 1 ? next++ : -1;
        if (faces) h.unit_of[6 * o + d] = unit[d];
      }
      for (int q = 0; q < 4; ++q) {  // pair q of the oct: y = q & 1, z = q >> 1
        const unsigned own = unsigned(8 * o + 2 * q - p.slot0);
        auto place = [&](int d, unsigned self, unsigned inside, unsigned cell) -> unsigned {
          if (unit[d] >= 0) return kResHalo | unsigned(4 * (unit[d] - p.unit0)) + cell;
          const int32_t nb = nbr[6 * o + d];
          return nb < 0 ? self : unsigned(8 * int64_t(nb) - p.slot0) + inside;
        };
        const int y = q & 1, z = q >> 1;
        const unsigned x0 = place(0, own, unsigned(2 * q + 1), unsigned(q));
        const unsigned x1 = place(1, own + 1, unsigned(2 * q), unsigned(q));
        const unsigned py = place(2 + y, own, unsigned(2 * (q ^ 1)), unsigned(2 * z));
        const unsigned pz = place(4 + z, own, unsigned(2 * (q ^ 2)), unsigned(2 * y));
        h.places[8 * o + 2 * q] = x0 | (x1 << 16);
        h.places[8 * o + 2 * q + 1] = py | (pz << 16);
      }
    }
    if (cnb) {
      const int32_t first = next;
      towards_finer(p, [&](int64_t i, int d, int32_t finer) {
        uint32_t& c = h.couplings[i >> 1];
        if (c == 0) c = uint32_t(next - first);
        c += i & 1 ? 1u << 24 : 1u << 16;
        h.coarse[2 * size_t(next)] = int32_t(i - p.slot0);
        h.coarse[2 * size_t(next) + 1] = 8 * finer + (d ^ 1);
        ++next;
      });
    }
  });
  h.partner.assign(n_units, -1);
  team.each(n_parts, [&](int k) {
    const ResPart& p = h.parts[k];
    for (int64_t o = oct0(p); o < oct1(p); ++o)
      for (int d = 0, u = unit0[o]; outer[o] >> d; ++d)
        if ((outer[o] >> d) & 1) {
          const int32_t nb = nbr[6 * o + d];
          if (nb >= 0) h.partner[u] = unit_of(6 * int64_t(nb) + (d ^ 1));
          ++u;
        }
    // (a finer oct's face towards a coarser leaf has that leaf's unit for its only partner)
    for (int32_t u = p.unit0 + p.n_units - p.n_coarse; u < p.unit0 + p.n_units; ++u) {
      const int32_t c = h.coarse[2 * size_t(u) + 1], f = unit_of(6 * int64_t(c >> 3) + (c & 7));
      h.partner[u] = f;
      h.partner[f] = u;
    }
  });
  h.n_near = ResPlanHost::near_base(n_units, n_parts);
  h.peers.resize(2 * size_t(n_units));
  team.each(n_parts, [&](int me) {
    const ResPart& mine = h.parts[me];
    for (int32_t u = mine.unit0; u < mine.unit0 + mine.n_units; ++u) {
      const int32_t k = share_of[h.partner[u]];
      const ResPart& p = h.parts[k];
      h.peers[2 * size_t(u)] = ResPlanHost::near_base(p.unit0, k) + (h.partner[u] - p.unit0);
      h.peers[2 * size_t(u) + 1] = k - p.part0;
    }
  });
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
