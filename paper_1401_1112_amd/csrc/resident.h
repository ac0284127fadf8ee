// Resident CG: the whole solve of a problem in one launch, its state in registers and
// LDS, one exchange of face values and partial sums between blocks per iteration.
#pragma once

#include <hip/hip_runtime.h>

#include <vector>

#include "device.h"
#include "resident_plan.h"

namespace amrfld {

constexpr int kResThreads = 512;
// Pairs of slots a thread holds with their coefficients, and the slots of a block then;
// larger shares, up to kResMaxSlots, read the coefficients in every iteration.
constexpr int kResPairs = 5;
constexpr int kResBlockSlots = 2 * kResPairs * kResThreads;
constexpr int kResMaxSlots = 16 * kResThreads;
constexpr int kResStreamDoubles = 11 * kResMaxSlots / 2;  // the coefficients of a block
constexpr int kResTargetSlots = 512;  // of one share where the level has several
// Polls (about a microsecond each) before a block gives up.  Once the blocks of a problem
// have met, in its first exchange, they wait for each other's arithmetic only, unless the
// device is taken from them as a whole.
constexpr unsigned kResSpinLoop = 1u << 22;
// Until then for the last one's place on the device, behind other streams' and processes'
// kernels: 0.3 s where the solve can be repeated in sweeps, which run beside them on what
// is left; as long as a grid barrier of the persistent sweeps where it cannot (captured
// steps, persistent batches).
constexpr unsigned kResSpinMeet = 1u << 18, kResSpinMeetFinal = 1u << 26;
// And for blocks that come from earlier patches of a batch: this many for each iteration
// that those may take (10 us of the largest shares).
constexpr unsigned kResPollsPerIteration = 16;
constexpr int kResWords = 7;  // a share's partial sums: words of 48 bits and a 16-bit stamp
constexpr int kResResumes = 4;  // launches after the first of a captured refined solve
constexpr int kResLine = 8;   // words of the line they lie in

// Device tables of a plan and its exchange memory.
struct ResPlanDev {
  const ResPart* parts = nullptr;
  const uint2* places = nullptr;  // per pair of slots: see ResPlanHost
  const int32_t* partner = nullptr;  // ResPlanHost::partner, then ::peers
  const int32_t* task0 = nullptr;
  const int32_t* task = nullptr;
  unsigned long long* lines = nullptr;  // [2][n_parts][kResLine]
  // [2][all_units()][4][2]: the units by their first number, padded to whole lines, where
  // the two shares run on different XCDs, then by their second where on the same
  unsigned long long* halo = nullptr;
  // [n_prob] next exchange number of each problem, advanced when its solve is complete;
  // [n_prob] that number once a block has begun to write the result of a solve; then the
  // flag of a wait that timed out
  unsigned* epoch = nullptr;
  // streamed coefficients, resident_coefs() of them; of a system with couplings between
  // levels (coupled) ResPlanHost::couplings, then ::coarse.  (One pointer and the sizes in
  // 32 bits: with larger arguments the compiler spills more of the loops.)
  void* extra = nullptr;
  int n_parts = 0, n_units = 0, n_prob = 0;
  int n_blocks = 0;
  int max_slots = 0;
  int lds = 0;  // bytes of LDS, resident_lds()
  int coupled = 0;
  int n_near = 0;

  __host__ __device__ int far_units() const { return (n_units + 1) & ~1; }
  __host__ __device__ int64_t all_units() const { return int64_t(far_units()) + n_near; }
};

struct ResArgs {
  const double* Cp = nullptr;    // assembled coefficients of the + faces
  const double* Cm = nullptr;    // and of the - faces
  const double* diag = nullptr;
  const double* b = nullptr;
  double* x = nullptr;           // x_0 on entry, the result on return
  PcgScalars* sc = nullptr;      // one record per problem, written whole
  double tol = 0.0, abs_floor = 0.0;
  int max_iter = 0, linf_test = 0, true_residual = 0;
  // refine (the mixed-precision form): segments that each reduce the residual by
  // inner_tol, max_outer of them at most, the stopping rule at their ends; the last one's
  // stop is decided on the true residual, and a solve that is still above its threshold is
  // resumed from its iterate by another launch (which does nothing where it is not).
  int refine = 0, resume = 0, max_outer = 0;
  double inner_tol = 0.0;
  // post-solve: T update of the coupling term
  CouplingParams cp{};
  const double* rho = nullptr;
  double* T_out = nullptr;
  double dt = 0.0;
  unsigned meet_limit = 0, spin_limit = 0;  // polls of a share's first exchange, of a later one
  // Of one problem, beside other launches: block b works on share b, and there is no other
  // block.  (Alone the shares lie on as few XCDs as hold them, which takes a grid over all of
  // them: 32 shares take 3.7 us an iteration so and 4.5 spread.)  The same bits either way.
  int spread = 0;
};

// Whether a block's share of this plan fits its registers and LDS.
bool resident_fits(const ResPlanDev& R);
int resident_lds(const std::vector<ResPart>& parts, int max_slots, int n_prob);
// Doubles of the streamed coefficients of a plan (0: none of its shares streams them).
size_t resident_coefs(const ResPlanDev& R);
// All blocks have to be on the device together (at most one per compute unit): no other
// kernel whose blocks wait for each other may run meanwhile, but for such as leave a unit
// for each block.  An ordinary launch: a cooperative one goes through a hardware queue of
// its own, which costs 20 to 130 us of waits between the queues on a solve of 300 us.
hipError_t launch_resident(hipStream_t s, const DevLevel& L, const ResPlanDev& R, const ResArgs& A);

}  // namespace amrfld
