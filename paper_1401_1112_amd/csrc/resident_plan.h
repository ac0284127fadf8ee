// How the octs of independent problems are dealt to the blocks of the resident CG
// (host side, no device code): contiguous shares of octs, and the faces between them.
#pragma once

#include <cstddef>
#include <cstdint>
#include <memory>
#include <utility>
#include <vector>

namespace amrfld {

constexpr unsigned kResHalo = 0x8000u;

// Entries that are not set when an array is made: a large plan is written by several
// threads, each of which so is the first to touch its part.
template <class T>
struct ResNoInit : std::allocator<T> {
  template <class U>
  struct rebind {
    typedef ResNoInit<U> other;
  };
  ResNoInit() = default;
  template <class U>
  ResNoInit(const ResNoInit<U>&) {}
  template <class U>
  void construct(U* p) {
    ::new (static_cast<void*>(p)) U;
  }
  template <class U, class... A>
  void construct(U* p, A&&... a) {
    ::new (static_cast<void*>(p)) U(std::forward<A>(a)...);
  }
};
template <class T>
using ResArray = std::vector<T, ResNoInit<T>>;

// One block's share of a problem: a contiguous range of its slots.
struct ResPart {
  int slot0, n_slots;  // its slots (whole octs)
  int unit0, n_units;  // its halo units: faces of its octs whose neighbour oct lies in another share
  int prob;            // the problem
  int part0, group;    // the problem's shares are [part0, part0 + group)
  int n_coarse;        // the last of its units: its cells' faces towards finer cells
};

// Where a share's arrays lie in LDS, in doubles from a 16-byte boundary: p^ and r^ of the
// slots and the halo, the exchanged values, the diagonal (held shares), the coefficients
// of the finer cells, and last the partner units, the only ones that are not read in pairs
// of 16 bytes.  cap: places of the slots (even).
struct ResLds {
  size_t p, rh, ex, diag, coarse, partner, bytes;
  constexpr ResLds(size_t cap, size_t units, size_t n_coarse, bool held)
      : p(0),
        rh(cap + 4 * units),
        ex(rh + 4 * units),
        diag(ex + 4 * units),
        coarse(diag + (held ? cap : 0)),
        partner(coarse + 4 * n_coarse),
        bytes(partner * sizeof(double) + ((units + 1) & ~size_t(1)) * sizeof(int32_t)) {}
};

struct ResPlanHost {
  std::vector<ResPart> parts;
  // unit_of[6 o + d]: number of the halo unit of oct o's face d, or -1 (where asked for).
  // Units are numbered share by share, so a share's units are contiguous.
  std::vector<int32_t> unit_of;
  // places[2 k], places[2 k + 1] of the slots 2 k and 2 k + 1, neighbours in x: where a
  // share's block finds their out-of-oct neighbours, 16 bits each.  Low and high half of
  // the first word: the neighbour in x of either slot; of the second: the pair of
  // neighbours in y, in z.  A position in the share, or kResHalo and a position among
  // its halo cells (four per unit); the slot or pair itself where there is none.
  ResArray<uint32_t> places;
  // partner[u]: the unit of the same face seen from the other side (the neighbour
  // share writes its four cells there)
  std::vector<int32_t> partner;
  // A second numbering of the units, each share's from a multiple of two on (two units
  // fill a cache line): share k's begin at near_base(unit0, k).
  static int32_t near_base(int32_t unit0, int32_t share) { return (unit0 + share + 1) & ~1; }
  int32_t n_near = 0;
  // peers[2 u], peers[2 u + 1]: the partner's number in it, and its share within the group
  std::vector<int32_t> peers;
  // Couplings between levels (empty: none).  A unit of a face towards a coarser leaf holds
  // that leaf's value four times and is an out-of-oct neighbour like any other.  A coarse
  // unit holds the four finer cells on one face of a leaf: coarse[2 u] is the leaf's
  // position in the share, coarse[2 u + 1] eight times the finer oct plus the direction
  // of its face.  couplings[k] of the slots 2 k and 2 k + 1: the first of their coarse
  // units (16 bits), the number of units of either (8 bits each), 0 where there is none.
  std::vector<int32_t> coarse;
  std::vector<uint32_t> couplings;
  // blocks: block b works on the shares task[task0[b] .. task0[b + 1]) in that order
  std::vector<int32_t> task0, task;
  int max_slots = 0, max_units = 0;  // of one share
};

// A problem's octs: [oct0, oct0 + n_oct) of the neighbour table; id: its scalar record.
struct ResProblem {
  int64_t oct0 = 0, n_oct = 0;
  int id = 0;
};

// Shares of a problem of n_oct octs: one where it fits a block (max_slots), else about
// target_slots each, at most max_blocks.  One block waits for nobody: 4096 slots take
// 2.5 us an iteration in one block and 3.5 in eight.  From two blocks on an iteration is
// the exchange (3 to 4 us) and 0.5 us per 1024 slots of a share; on one XCD the exchange
// is cheap enough for small shares: 16 k slots take 4.0 us in 16 blocks and 3.7 in 32
// (4.5 in 16 spread over the XCDs), 88 k slots 5.2 us in 88 and 5.1 in 176.
int res_group(int64_t n_oct, int max_blocks, int max_slots, int target_slots);

// Blocks to launch for one problem in g shares on n_cu compute units of 8 XCDs, to which
// blocks are dealt round-robin: as many as it takes for its shares to lie on as few XCDs
// as hold them (the other blocks have no share and end at once).
int res_blocks(int g, int n_cu);

// About what an iteration of a share of n_slots slots takes in a group (us).
double res_cost(int n_slots, int group);

// Plans problems (listed in the order the blocks work on them) on n_blocks blocks;
// group[q] shares of problem q, all on different blocks.  nbr: 6 per oct, as in
// LevelTables (the neighbour of o in direction d has o as its neighbour in d ^ 1).
// n_oct_table: rows of nbr.  cnb, child (not null: a system with couplings between levels):
// the coarser leaf behind each face without a neighbour oct, -1 where there is none; the
// oct that refines each slot, negative where there is none, -1 where the slot is a leaf.
// faces: unit_of as well.  threads: 0 for one per kResPlanThreadOcts octs, at most
// kResPlanThreads; the plan is the same whatever their number.  Two million octs take 126 ms
// in one thread, 48 in four and 36 in eight; for 40 thousand (2 ms) starting threads costs
// what they save.
constexpr int64_t kResPlanThreads = 8, kResPlanThreadOcts = 65536;
ResPlanHost build_res_plan(const std::vector<ResProblem>& probs, const std::vector<int>& group, int n_blocks,
                           const int32_t* nbr, int64_t n_oct_table, const int32_t* cnb = nullptr,
                           const int32_t* child = nullptr, bool faces = true, int threads = 0);

}  // namespace amrfld
