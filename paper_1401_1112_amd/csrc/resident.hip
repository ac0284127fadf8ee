// Resident CG (Sect. 3.3.4): see resident.h.
//
// A block holds a contiguous share of a problem's slots for the whole solve: the scaled
// face coefficients, the iterate, the residual and s^ = A^ p^ in registers, the search
// direction p^ and the diagonal in LDS.  Nothing of the system is read from memory again
// after the start.  Between blocks an iteration exchanges only the s^ of the cells on
// faces between shares (each block keeps copies of its outer neighbours' r^ and p^ and
// updates them with the arithmetic of their owner, so the copies are the owner's bits)
// and four partial sums per share.
//
// A thread holds pairs of slots that are neighbours in x, four threads an oct: the
// sibling in x is the thread's own, those in y and z come by quad permutes, and the
// out-of-oct neighbours in y and z of both slots are one 16-byte LDS read.
//
// The recurrences are those of CG on the Jacobi-scaled system with one reduction per
// iteration: s^_k = A^ p^_k, alpha_k = (r^,r^) / (p^,s^), and the next residual norm
// that beta_k needs is formed from the sums of the same exchange,
//   (r^_{k+1}, r^_{k+1}) = alpha^2 (s^,s^) - (r^,r^)
// ((r^,s^) = (p^,s^), p^ being conjugate to its predecessor), while
// (r^_{k+1}, r^_{k+1}) itself is summed with the next exchange and used for alpha_{k+1}:
// the step along p^ stays a line search, and no error is carried on.
//
// The composite system of several levels: a finer cell's face towards a coarser leaf is
// an out-of-oct face like any other, its halo cell the leaf's value; a leaf's face
// towards finer cells is a unit with their four values, added to its row by its thread
// with coefficients from LDS.  All couplings go through the exchange, also those within
// a share.  Four levels of 353 k slots, 400 iterations in four solves: 13.1 ms with
// sweeps and a kernel for the couplings, 4.1 so (8.3 us per iteration: shares of 1400
// slots have 207 to 658 units, as many as shares of 4880 slots of one level).
//
// Every exchanged word carries the number of its exchange (a 64-bit word holds data
// and stamp), so a reader polls the data itself: no barrier, no flag after the data and
// no cache write-back stand between a value's store and its use.  Two buffers
// alternate: a block stores into a buffer again only after it has seen every block's
// sums of the exchange between, and so after every block has read it.  Every wait is
// bounded; a block that gives up sets the abort flag and leaves, the others then time
// out in turn, and the iterate in memory is untouched.  While the flag is set the
// exchange numbers are those of the launch that gave up, and its words may still be
// there: until the host has cleared the exchange, a share of several ends at its first
// exchange.  A problem's record has its done flag set only by a launch that completed it.
#include "resident.h"

#include <algorithm>

#include "common.h"

namespace amrfld {

namespace {

typedef unsigned long long u64;

constexpr int kWaves = kResThreads / 64;
constexpr int kSums = 4;
constexpr int kMaxShares = kResThreads;  // of a problem: a thread reads the words of one
constexpr double kUnderflow = 1e-290;  // sums of squares below it are short of bits
constexpr u64 kMask48 = 0xffffffffffffull;

__device__ __forceinline__ u64 ld_word(const u64* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// A store that only this XCD has to see: into its L2, which agent-scope loads on the XCD
// read as well, and no further.
__device__ __forceinline__ void st_word_near(u64* p, u64 v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ unsigned xcc_id() { return __builtin_amdgcn_s_getreg(20 | (0 << 6) | (3 << 11)); }
__device__ __forceinline__ void st_word(u64* p, u64 v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_word32(unsigned* p, unsigned v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ u64 bits_of(double v) { return u64(__double_as_longlong(v)); }
__device__ __forceinline__ double of_bits(u64 w) { return __longlong_as_double((long long)w); }
__device__ __forceinline__ double of_words(unsigned lo, unsigned hi) { return of_bits((u64(hi) << 32) | lo); }

// The thread's number, recomputed where it is used: addresses derived from it are not
// kept in registers from one phase to the next.
__device__ __forceinline__ int tid() {
  int t = int(threadIdx.x);
  asm volatile("" : "+v"(t));
  return t;
}

// The value is formed here: not later, where its inputs would have to be kept as well.
template <typename T>
__device__ __forceinline__ void keep(T& v) {
  asm volatile("" : "+v"(v));
}

// v of the lane that kCtrl names, `old` where there is none.
template <int kCtrl>
__device__ __forceinline__ double dpp(double old, double v) {
  const u64 w = bits_of(v), o = bits_of(old);
  return of_words(
      unsigned(__builtin_amdgcn_update_dpp(int(unsigned(o)), int(unsigned(w)), kCtrl, 0xf, 0xf, false)),
      unsigned(__builtin_amdgcn_update_dpp(int(unsigned(o >> 32)), int(unsigned(w >> 32)), kCtrl, 0xf, 0xf, false)));
}
constexpr int kQuadXor1 = 0xB1, kQuadXor2 = 0x4E, kRowShr1 = 0x111, kRowShr2 = 0x112, kRowShr4 = 0x114,
              kRowShr8 = 0x118;

// a + b after the upper half wave of a has changed places with the lower half of b: a
// summed over lane pairs 32 apart in the lower half, b in the upper half.
__device__ __forceinline__ double fold32(double a, double b) {
  const u64 x = bits_of(a), y = bits_of(b);
  const auto lo = __builtin_amdgcn_permlane32_swap(unsigned(x), unsigned(y), false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap(unsigned(x >> 32), unsigned(y >> 32), false, false);
  return of_words(lo[0], hi[0]) + of_words(lo[1], hi[1]);
}
// The same with the odd rows of 16 lanes of a and the even rows of b.
__device__ __forceinline__ double fold16(double a, double b) {
  const u64 x = bits_of(a), y = bits_of(b);
  const auto lo = __builtin_amdgcn_permlane16_swap(unsigned(x), unsigned(y), false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(unsigned(x >> 32), unsigned(y >> 32), false, false);
  return of_words(lo[0], hi[0]) + of_words(lo[1], hi[1]);
}
// Wave-wide sums of four values: the last lane of row 0, 1, 2, 3 returns that of v[0],
// v[2], v[1], v[3].  Folding halves the values with the lanes: 7 additions, not 24.
__device__ __forceinline__ double wave_sums(const double (&v)[kSums]) {
  double a = fold16(fold32(v[0], v[1]), fold32(v[2], v[3]));
  a += dpp<kRowShr1>(0.0, a);
  a += dpp<kRowShr2>(0.0, a);
  a += dpp<kRowShr4>(0.0, a);
  a += dpp<kRowShr8>(0.0, a);
  return a;
}
__device__ __forceinline__ double wave_max(double a) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) a = fmax(a, __shfl_xor(a, o, 64));
  return a;
}

// LDS of a block.
struct Shared {
  double part[kWaves][kSums + 1];   // per wave: this share's sums and maximum
  double total[kWaves][kSums + 1];  // per wave: over the shares' words
  double gate[kWaves];  // per wave (its lanes alone read and write it): cg_loop's gate
  int failed;
  unsigned char xcc[kMaxShares];  // where the problem's shares run, from the first exchange on
};

struct Exchange {
  const ResPlanDev& R;
  const ResPart& me;
  int my_part;
  unsigned epoch;  // number of the next exchange
  unsigned near;  // bit k: this thread's k-th word of the halo is among the near ones
  bool one_xcd;   // all shares of the only problem run on one XCD

  // the words of share `part`: a 64-byte line that one store fills
  __device__ __forceinline__ u64* words(int part) const {
    return R.lines + (size_t(epoch & 1u) * R.n_parts + part) * kResLine;
  }
  __device__ __forceinline__ u64* halo(int unit) const {
    return R.halo + (size_t(epoch & 1u) * R.all_units() + unit) * 8;
  }
};

// The arguments of a kernel, read from the launch's memory again wherever this is called.
// Taken as parameters they are read once, at the start, and what is used after the
// iterations is moved out of the way and back within them: 146 such moves of a lane in the
// loop of shares of 1024 slots, 44 so.  An iteration of 4096 slots in one block takes
// 1.99 us for 2.08, of 33 k slots in 64 blocks 3.4 for 3.5, of 262 k in 256 4.25 for 4.45,
// two steps of 64 patches (16.8 M slots) 40.8 ms for 43.0.
struct KernelArgs {
  DevLevel L;
  ResPlanDev R;
  ResArgs A;
};
typedef const __attribute__((address_space(4))) char* ArgMemory;
// (read as what it is, a pointer to device memory, which the compiler takes for granted of
// arguments that it reads itself)
template <class T>
__device__ __forceinline__ void read_pointer(ArgMemory a, size_t at, T*& p) {
  typedef __attribute__((address_space(1))) T* Global;
  p = (T*)*(const __attribute__((address_space(4))) Global*)(a + at);
}
__device__ __forceinline__ KernelArgs kernel_args() {
  ArgMemory a = (ArgMemory)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(a));
  KernelArgs k;
#pragma unroll
  for (int i = 0; i < int(sizeof(KernelArgs) / sizeof(int)); ++i)
    reinterpret_cast<int*>(&k)[i] = ((const __attribute__((address_space(4))) int*)a)[i];
#define AMRFLD_POINTER(f) read_pointer(a, offsetof(KernelArgs, f), k.f)
  AMRFLD_POINTER(L.child);
  AMRFLD_POINTER(L.cif);
  AMRFLD_POINTER(R.parts);
  AMRFLD_POINTER(R.places);
  AMRFLD_POINTER(R.partner);
  AMRFLD_POINTER(R.task0);
  AMRFLD_POINTER(R.task);
  AMRFLD_POINTER(R.lines);
  AMRFLD_POINTER(R.halo);
  AMRFLD_POINTER(R.epoch);
  AMRFLD_POINTER(R.extra);
  AMRFLD_POINTER(A.Cp);
  AMRFLD_POINTER(A.Cm);
  AMRFLD_POINTER(A.diag);
  AMRFLD_POINTER(A.b);
  AMRFLD_POINTER(A.x);
  AMRFLD_POINTER(A.sc);
  AMRFLD_POINTER(A.cp.T);
  AMRFLD_POINTER(A.rho);
  AMRFLD_POINTER(A.T_out);
#undef AMRFLD_POINTER
  return k;
}

// Words of one value in the halo memory, and of the four of a unit.
constexpr int kValueWords = 2, kUnitWords = 4 * kValueWords;

__device__ __forceinline__ unsigned half(double v, int h) { return unsigned(bits_of(v) >> (32 * h)); }

// The export list to the partners' halo memory: consecutive lanes store consecutive
// words, so that one store fills a unit's line.  Units whose partner runs on the same XCD
// lie past far_units() and stay in its L2: 256 blocks that exchange 340 units each take
// 3.0 us so and 5.7 through memory, 600 units 3.4 and 7.2.  (The two kinds never share a
// cache line, nor do near units of two shares: a line is written from one XCD only.)
// A step of four levels to 1.25 M slots: 12.1 ms with all units through memory, 10.9 so.
__device__ __forceinline__ void put_halo(const Exchange& X, const double* ex, const int* partner) {
  const u64 st = u64(X.epoch) << 32;
  u64* const h = X.halo(0);
  const int far = X.R.far_units();
  constexpr int kBatch = 4;  // words of a thread at a time, so that their LDS reads overlap
  const int nw = kUnitWords * X.me.n_units;
  for (int w0 = tid(); w0 < nw; w0 += kBatch * kResThreads) {
    int to[kBatch];
    unsigned d[kBatch];
#pragma unroll
    for (int k = 0; k < kBatch; ++k) {
      const int w = min(w0 + k * kResThreads, nw - 1);
      to[k] = partner[w / kUnitWords];
      d[k] = half(ex[w / kValueWords], w % kValueWords);
    }
#pragma unroll
    for (int k = 0; k < kBatch; ++k) {
      u64* const p = h + (size_t(to[k]) * 8 + w0 % kUnitWords);
      if (w0 + k * kResThreads >= nw) break;
      if (to[k] >= far) st_word_near(p, st | d[k]);
      else st_word(p, st | d[k]);
    }
  }
}

// The halo values of this exchange to sh, a word per lane, kBatch words of a thread in
// flight.  Every value is stored by the thread that exported the one at the same place,
// so sh and ex are the same memory.  false: a wait timed out.
template <int kBatch>
__device__ __forceinline__ bool get_halo(const Exchange& X, unsigned limit, double* sh) {
  const int nw = kUnitWords * X.me.n_units;
  const u64* h = X.halo(X.me.unit0);
  // from a unit's place among the far ones to that among the near ones (near_base)
  const unsigned to_near = 8u * unsigned(X.R.far_units() + ((X.me.unit0 + X.my_part + 1) & ~1) - X.me.unit0);
  unsigned polls = 0, near = X.near;
  for (int w0 = tid(); w0 < nw; w0 += kBatch * kResThreads) {
    u64 c[kBatch];
    // (a lane past the end polls the last word, so no lane is masked)
    auto word = [&](int k) {
      return ld_word(h + (unsigned(min(w0 + k * kResThreads, nw - 1)) + ((0u - ((near >> k) & 1u)) & to_near)));
    };
#pragma unroll
    for (int k = 0; k < kBatch; ++k) c[k] = word(k);
    for (;;) {  // words that are not there yet are read again, and no others
      asm volatile("" : "+v"(near));  // (no masks kept from one round to the next)
      unsigned missing = 0;
#pragma unroll
      for (int k = 0; k < kBatch; ++k) {
        const unsigned miss = unsigned(c[k] >> 32) ^ X.epoch;
        missing |= miss;
        if (miss) c[k] = word(k);
      }
      if (!missing) break;
      if (++polls > limit) return false;
    }
#pragma unroll
    for (int k = 0; k < kBatch; ++k) {
      const int w = w0 + k * kResThreads;
      const unsigned mine = unsigned(c[k]);
      // the other half is in the neighbour lane
      const unsigned other = unsigned(__builtin_amdgcn_update_dpp(0, int(mine), kQuadXor1, 0xf, 0xf, false));
      if (w < nw && !(w & 1)) sh[w >> 1] = of_words(mine, other);
    }
    near >>= kBatch;
  }
  return true;
}
__device__ __forceinline__ bool get_halo(const Exchange& X, unsigned limit, double* sh) {
  const int nw = kUnitWords * X.me.n_units;
  if (nw <= 2 * kResThreads) return get_halo<2>(X, limit, sh);
  if (nw <= 4 * kResThreads) return get_halo<4>(X, limit, sh);
  return get_halo<8>(X, limit, sh);
}

// The sums (k < kSums) and the maximum over the first n of the waves' rows, the same in
// every thread: lanes 8 k .. 8 k + 7 hold value k of the rows and add them up.
__device__ __forceinline__ void row_totals(const double (&rows)[kWaves][kSums + 1], int n, bool wide,
                                           double (&v)[kSums], double& m) {
  const int lane = tid() & 63;
  const bool in = (lane & 7) < n;
  double c = lane < 8 * kSums && in ? rows[lane & 7][lane >> 3] : 0.0;
  c += dpp<kRowShr1>(0.0, c);
  c += dpp<kRowShr2>(0.0, c);
  c += dpp<kRowShr4>(0.0, c);
  const u64 w = bits_of(c);
#pragma unroll
  for (int k = 0; k < kSums; ++k)
    v[k] = of_words(unsigned(__builtin_amdgcn_readlane(int(unsigned(w)), 8 * k + 7)),
                    unsigned(__builtin_amdgcn_readlane(int(unsigned(w >> 32)), 8 * k + 7)));
  if (wide) {
    double x = in ? rows[lane & 7][kSums] : -DBL_MAX;
    x = fmax(x, dpp<kRowShr1>(x, x));
    x = fmax(x, dpp<kRowShr2>(x, x));
    x = fmax(x, dpp<kRowShr4>(x, x));
    const u64 e = bits_of(x);
    m = of_words(unsigned(__builtin_amdgcn_readlane(int(unsigned(e)), 7)),
                 unsigned(__builtin_amdgcn_readlane(int(unsigned(e >> 32)), 7)));
  }
}

// This share's sums v and (wide) maximum m published, and its export list ex (null:
// none); a problem of one share: the sums returned to every thread.
__device__ __forceinline__ void put_sums(const Exchange& X, double (&v)[kSums], double& m, bool wide, Shared& S,
                                         const double* ex, const int* partner) {
  const int t = tid(), lane = t & 63, wid = t >> 6;
  const double a = wave_sums(v);
  if ((lane & 15) == 15) S.part[wid][((lane >> 5) & 1) | ((lane >> 3) & 2)] = a;
  if (wide) {
    const double b = wave_max(m);
    if (lane == 0) S.part[wid][kSums] = b;
  }
  __syncthreads();
  if (X.me.group == 1) {
    row_totals(S.part, kWaves, wide, v, m);
    __syncthreads();
    return;
  }
  if (ex) put_halo(X, ex, partner);
  if (wid == 0) {
    double x = 0.0;
    row_totals(S.part, kWaves, wide, v, x);
    const u64 d0 = bits_of(v[0]), d1 = bits_of(v[1]), d2 = bits_of(v[2]), d3 = bits_of(v[3]), e = bits_of(x);
    // 48 bits of data to a word
    u64 word = d0;
    word = lane == 1 ? (d0 >> 48) | (d1 << 16) : word;
    word = lane == 2 ? (d1 >> 32) | (d2 << 32) : word;
    word = lane == 3 ? d2 >> 16 : word;
    word = lane == 4 ? d3 : word;
    word = lane == 5 ? (d3 >> 48) | (e << 16) : word;
    word = lane == 6 ? (e >> 32) | (u64(xcc_id()) << 32) : word;
    word = (word & kMask48) | (u64(X.epoch & 0xffffu) << 48);
    // (also the last word, which is read with the maximum only: its stamp of 16 bits then
    // differs from any that is awaited, however many exchanges lie between two maxima)
    if (lane < kResWords) {
      if (X.one_xcd) st_word_near(X.words(X.my_part) + lane, word);
      else st_word(X.words(X.my_part) + lane, word);
    }
  }
}

// The sums (and maximum) over the whole problem to every thread, and the halo values
// that the neighbour shares published for this exchange to sh (null: none).  false: a
// wait took more than limit polls.
__device__ __forceinline__ bool collect(Exchange& X, unsigned limit, double (&v)[kSums], double& m, bool wide, Shared& S,
                                        double* sh) {
  const int t = tid(), lane = t & 63, wid = t >> 6, G = X.me.group;
  if (G == 1) {
    ++X.epoch;
    return true;
  }
  const int n_waves = (G + 63) >> 6;
  bool ok = !sh || get_halo(X, limit, sh);
  if (wid < n_waves) {
    u64 w[kResWords];
#pragma unroll
    for (int k = 0; k < kResWords; ++k) w[k] = 0;
    if (t < G && ok) {
      const unsigned st = X.epoch & 0xffffu;
      const u64* ln = X.words(X.me.part0 + t);
      unsigned polls = 0;
      for (;;) {
        bool all = true;
#pragma unroll
        for (int k = 0; k < kResWords; ++k)
          if (k < kResWords - 1 || wide) w[k] = ld_word(ln + k);
#pragma unroll
        for (int k = 0; k < kResWords; ++k)
          if (k < kResWords - 1 || wide) all = all && unsigned(w[k] >> 48) == st;
        if (all) break;
        if (++polls > limit) {
          ok = false;
          break;
        }
      }
#pragma unroll
      for (int k = 0; k < kResWords; ++k) w[k] &= kMask48;
    }
    v[0] = of_bits(w[0] | (w[1] << 48));
    v[1] = of_bits((w[1] >> 16) | (w[2] << 32));
    v[2] = of_bits((w[2] >> 32) | (w[3] << 16));
    v[3] = of_bits(w[4] | (w[5] << 48));
    const double a = wave_sums(v);
    if ((lane & 15) == 15) S.total[wid][((lane >> 5) & 1) | ((lane >> 3) & 2)] = a;
    if (wide) {
      if (t < G) S.xcc[t] = (unsigned char)(w[6] >> 32);
      const double b = wave_max(t < G ? of_bits((w[5] >> 16) | (w[6] << 32)) : -DBL_MAX);
      if (lane == 0) S.total[wid][kSums] = b;
    }
  }
  if (!ok) S.failed = 1;
  __syncthreads();
  row_totals(S.total, n_waves, wide, v, m);
  ++X.epoch;
  return S.failed == 0;
}


// Scaled face coefficients of a pair: within the oct cix (the same for both slots), ciy,
// ciz; out of the oct cox, coy, coz.
struct Coefs {
  double cix, ciy[2], ciz[2], cox[2], coy[2], coz[2];
};

// A share's state in registers, NP pairs of slots per thread (thread t holds pairs
// t + 512 u of the share).  Places in p: of the out-of-oct neighbours in x of both slots
// (px, 16 bits each) and of the pairs in y and z (pyz).
template <int NP>
struct State {
  double x[NP][2], r[NP][2], s[NP][2];
  unsigned px[NP], pyz[NP];
  unsigned face;  // bit u: pair u has a cell on a face between shares
};

// What a share's loops hold where.
enum ResMode { kHeld, kStreamed, kCoupled };

// With the coefficients in registers too and the diagonal in LDS, or (kStreamed: shares of
// more than 5120 slots, whose coefficients do not fit) with the diagonal in registers and
// the coefficients read in every iteration, from memory that this block alone uses: 44
// bytes per slot that L2 and the last-level cache largely hold, against the 115 of a
// sweep.  What ends it at 8192 slots is the register file.  64 patches of 16.9 M cells,
// the 7.8 M of five of them in streamed shares (128^3 and less): 40 ms for two steps
// against 69 with sweeps of those five.
template <int NP, ResMode kMode>
struct Regs;

template <int NP>
struct Regs<NP, kHeld> : State<NP> {
  Coefs c[NP];
  double* d;

  __device__ __forceinline__ Coefs coefs(int u) const { return c[u]; }
  __device__ __forceinline__ void put_axis(int u, int a, double ci0, double ci1, double co0, double co1) {
    double(&ci)[2] = a == 1 ? c[u].ciy : c[u].ciz;
    double(&co)[2] = a == 0 ? c[u].cox : a == 1 ? c[u].coy : c[u].coz;
    if (a == 0) {
      c[u].cix = ci0;
      keep(c[u].cix);
    } else {
      ci[0] = ci0;
      ci[1] = ci1;
      keep(ci[0]);
      keep(ci[1]);
    }
    co[0] = co0;
    co[1] = co1;
    keep(co[0]);
    keep(co[1]);
  }
  __device__ __forceinline__ double2 diag(int u) const {
    return *reinterpret_cast<const double2*>(d + 2 * (tid() + u * kResThreads));
  }
  __device__ __forceinline__ void put_diag(int u, double2 v) {
    *reinterpret_cast<double2*>(d + 2 * (tid() + u * kResThreads)) = v;
  }
};

template <int NP>
struct Regs<NP, kStreamed> : State<NP> {
  double dr[NP][2];
  double2* cs;  // five arrays of NP * 512 pairs (ciy, ciz, cox, coy, coz), then cix

  __device__ __forceinline__ double2* at(int k, int u) const { return cs + (k * NP + u) * kResThreads + tid(); }
  __device__ __forceinline__ double* x_at(int u) const {
    return reinterpret_cast<double*>(cs + 5 * NP * kResThreads) + u * kResThreads + tid();
  }
  __device__ __forceinline__ Coefs coefs(int u) const {
    const double2 iy = *at(0, u), iz = *at(1, u), ox = *at(2, u), oy = *at(3, u), oz = *at(4, u);
    return Coefs{*x_at(u), {iy.x, iy.y}, {iz.x, iz.y}, {ox.x, ox.y}, {oy.x, oy.y}, {oz.x, oz.y}};
  }
  __device__ __forceinline__ void put_axis(int u, int a, double ci0, double ci1, double co0, double co1) {
    if (a == 0) *x_at(u) = ci0;
    else *at(a - 1, u) = double2{ci0, ci1};
    *at(2 + a, u) = double2{co0, co1};
  }
  __device__ __forceinline__ double2 diag(int u) const { return double2{dr[u][0], dr[u][1]}; }
  __device__ __forceinline__ void put_diag(int u, double2 v) {
    dr[u][0] = v.x;
    dr[u][1] = v.y;
    keep(dr[u][0]);
    keep(dr[u][1]);
  }
};

// As kHeld, and couplings to finer cells.
template <int NP>
struct Regs<NP, kCoupled> : Regs<NP, kHeld> {
  unsigned cu[NP];  // of a pair: first of its coarse units (16 bits), units of either slot (8 bits each)
  double* cv;       // [4 coarse units]: scaled coefficients of their finer cells (in LDS)
  int uc0;          // halo position of the first coarse unit
};

// LDS arrays of a share.
struct Lds {
  double* p;    // [cap + 4 units]: p^ of the share, then of its halo cells
  double* rh;   // [4 units]: r^ of the halo cells
  double* ex;   // [4 units]: this share's cells on the same faces, then the halo cells'
                // values of the current exchange
  int* partner; // [units]
};

// (A^ v) of pair u, v in p.
template <int NP>
__device__ __forceinline__ void apply(const State<NP>& q, const Coefs& c, const double* p, int u, double (&pv)[2],
                                      double (&av)[2]) {
  const int l = 2 * (tid() + u * kResThreads);
  const double2 own = *reinterpret_cast<const double2*>(p + l);
  const double2 ny = *reinterpret_cast<const double2*>(p + (q.pyz[u] & 0xffffu));
  const double2 nz = *reinterpret_cast<const double2*>(p + (q.pyz[u] >> 16));
  const double nx0 = p[q.px[u] & 0xffffu], nx1 = p[q.px[u] >> 16];
  pv[0] = own.x;
  pv[1] = own.y;
  double a0 = own.x, a1 = own.y;
  a0 = fma(-c.cix, own.y, a0);
  a1 = fma(-c.cix, own.x, a1);
  a0 = fma(-c.ciy[0], dpp<kQuadXor1>(own.x, own.x), a0);
  a1 = fma(-c.ciy[1], dpp<kQuadXor1>(own.y, own.y), a1);
  a0 = fma(-c.ciz[0], dpp<kQuadXor2>(own.x, own.x), a0);
  a1 = fma(-c.ciz[1], dpp<kQuadXor2>(own.y, own.y), a1);
  a0 = fma(-c.cox[0], nx0, a0);
  a1 = fma(-c.cox[1], nx1, a1);
  a0 = fma(-c.coy[0], ny.x, a0);
  a1 = fma(-c.coy[1], ny.y, a1);
  a0 = fma(-c.coz[0], nz.x, a0);
  a1 = fma(-c.coz[1], nz.y, a1);
  av[0] = a0;
  av[1] = a1;
}

// f(u, v, A^ v) for every pair; streamed coefficients are loaded one pair ahead.
template <int NP, ResMode kMode, class F>
__device__ __forceinline__ void apply_all(const Regs<NP, kMode>& q, const double* p, F f) {
  Coefs c = q.coefs(0);
#pragma unroll
  for (int u = 0; u < NP; ++u) {
    __builtin_amdgcn_sched_barrier(0);
    Coefs next;
    if (kMode == kStreamed && u + 1 < NP) next = q.coefs(u + 1);
    double pv[2], av[2];
    apply(q, c, p, u, pv, av);
    if constexpr (kMode == kCoupled) {
      if (q.cu[u]) {
        const int k1 = int(q.cu[u] & 0xffffu) + int((q.cu[u] >> 16) & 0xffu), k2 = k1 + int(q.cu[u] >> 24);
        const double* ph = p + 2 * NP * kResThreads + q.uc0;
        for (int k = int(q.cu[u] & 0xffffu); k < k2; ++k) {
          double t = 0.0;
#pragma unroll
          for (int e = 0; e < 4; ++e) t = fma(q.cv[4 * k + e], ph[4 * k + e], t);
          if (k < k1) av[0] -= t;
          else av[1] -= t;
        }
      }
    }
    f(u, pv, av);
    if (u + 1 < NP) c = kMode == kStreamed ? next : q.coefs(u + 1);
  }
}

// The values of pair u that lie on faces between shares to the block's export list
// (ordered like its halo cells).
template <int NP, ResMode kMode>
__device__ __forceinline__ void stage(const Regs<NP, kMode>& q, double* ex, int u, double v0, double v1) {
  constexpr int kCap = 2 * NP * kResThreads;
  if constexpr (kMode == kCoupled) {
    if (q.cu[u]) {
      const int k1 = int(q.cu[u] & 0xffffu) + int((q.cu[u] >> 16) & 0xffu), k2 = k1 + int(q.cu[u] >> 24);
      for (int k = int(q.cu[u] & 0xffffu); k < k2; ++k)
#pragma unroll
        for (int e = 0; e < 4; ++e) ex[q.uc0 + 4 * k + e] = k < k1 ? v0 : v1;
    }
  }
  if (!((q.face >> u) & 1u)) return;
  const int x0 = int(q.px[u] & 0xffffu) - kCap, x1 = int(q.px[u] >> 16) - kCap;
  const int y = int(q.pyz[u] & 0xffffu) - kCap, z = int(q.pyz[u] >> 16) - kCap;
  if (x0 >= 0) ex[x0] = v0;
  if (x1 >= 0) ex[x1] = v1;
  double2 w;
  w.x = v0;
  w.y = v1;
  if (y >= 0) *reinterpret_cast<double2*>(ex + y) = w;
  if (z >= 0) *reinterpret_cast<double2*>(ex + z) = w;
}

__device__ __forceinline__ bool exchange(Exchange& X, unsigned limit, double (&v)[kSums], double& m, bool wide,
                                         Shared& S, const Lds& lds) {
  put_sums(X, v, m, wide, S, lds.ex, lds.partner);
  return collect(X, limit, v, m, wide, S, lds.ex);
}

struct CgResult {
  double rn, linf;
  int iters, segments;
  bool fin, conv;
};

// CG iterations from r^ = q.r, p^ in lds.p (own and halo), r^ of the halo in lds.rh.
// thresh, tol, max_iter, linf_test: the stopping rule of Sect. 3.3.4; dmin: smallest
// diagonal entry.  The rule is looked at where ||r||^2 <= S.gate.  A refined solve: only
// there, where a segment ends, and the next one, of max_segments at most, ends where ||r||
// has fallen by A.inner_tol again, so that the last residual lies as far below the
// threshold as that of the refinement with FP32 segments.  false: a wait timed out.
template <int NP, ResMode kMode>
__device__ __forceinline__ bool cg_loop(Exchange& X, Regs<NP, kMode>& q, const Lds& lds, Shared& S, double thresh,
                                        double tol, int max_iter, bool linf_test, double dmin, const ResArgs& A,
                                        int max_segments, CgResult& out) {
  constexpr int kCap = 2 * NP * kResThreads;
  const int nh = 4 * X.me.n_units;
  double rr = 0.0, rrd = 0.0, linf = 0.0;
#pragma unroll
  for (int u = 0; u < NP; ++u) {
    const double2 d = q.diag(u);
    const double a0 = q.r[u][0] * q.r[u][0], a1 = q.r[u][1] * q.r[u][1];
    rr += a0 + a1;
    rrd = fma(a0, d.x, fma(a1, d.y, rrd));
  }
  bool wide = false;  // the next exchange carries the largest relative change too
  bool last = A.refine && max_segments <= 1;  // no segment after this one
  for (int k = 0;; ++k) {
    double v[kSums] = {0.0, 0.0, rr, rrd};
    // (opaque: nothing derived from the places is kept in registers across iterations)
#pragma unroll
    for (int u = 0; u < NP; ++u) asm volatile("" : "+v"(q.px[u]), "+v"(q.pyz[u]));
    apply_all(q, lds.p, [&](int u, const double(&pv)[2], const double(&av)[2]) {
      q.s[u][0] = av[0];
      q.s[u][1] = av[1];
      stage(q, lds.ex, u, av[0], av[1]);
      v[0] = fma(pv[0], av[0], fma(pv[1], av[1], v[0]));
      v[1] = fma(av[0], av[0], fma(av[1], av[1], v[1]));
    });
    const double gate = S.gate[tid() >> 6];
    if (!exchange(X, A.spin_limit, v, linf, wide, S, lds)) return false;
    // the stopping test of iterate k
    if (k >= 1) {
      // (the root only where it can matter: it is a long chain before alpha)
      out.fin = isfinite(v[3]) && isfinite(v[0]) && isfinite(v[2]);
      if (!out.fin || v[3] <= gate || k >= max_iter) {
        out.rn = sqrt(v[3]);
        out.linf = linf;
        out.iters = k;
        out.conv = out.fin && ((out.rn <= thresh && (!linf_test || (wide && linf < tol))) || out.rn == 0.0);
        if (A.refine) {
          if (++out.segments >= max_segments) return true;
          S.gate[tid() >> 6] = A.inner_tol * A.inner_tol * v[3];
          last = out.segments + 1 >= max_segments;
        }
        if (!out.fin || out.conv || k >= max_iter) return true;
      }
    }
    // alpha = gam / (p^,s^); beta = (alpha^2 (s^,s^) - gam) / gam
    const double gam = v[2];
    const double inv = 1.0 / v[0];
    double alpha = gam * inv, ratio = fma(alpha * inv, v[1], -1.0);
    if (!isfinite(alpha) || !isfinite(ratio)) {
      // the inverse overflows before the quotients do
      alpha = gam / v[0];
      ratio = fma(alpha, v[1] / v[0], -1.0);
      if (!isfinite(alpha) || !isfinite(ratio)) {
        out.rn = sqrt(v[3]);
        out.linf = 0.0;
        out.iters = k;
        ++out.segments;
        // a residual below its threshold whose squares underflow is zero (cells that a
        // pulse has barely reached keep the relative change above tol until then)
        out.fin = out.conv = k >= 1 && v[0] == 0.0 && gam < kUnderflow && (out.rn <= thresh || thresh == 0.0);
        return true;
      }
    }
    const double beta = ratio > 0.0 ? ratio : 0.0;
    const double gnext = beta * gam;
    // ||r_{k+1}||^2 >= dmin (r^,r^)_{k+1}: where that is above the threshold (with a
    // margin for the rounding of the prediction) iterate k + 1 cannot be the last, and its
    // relative change, a division per cell, is not formed (the last segment that a
    // refined solve may make ends the solve whatever its residual)
    wide = last || k + 1 >= max_iter || !(gnext * dmin > 4.0 * thresh * thresh);
    rr = rrd = linf = 0.0;
#pragma unroll
    for (int u = 0; u < NP; ++u) {
      __builtin_amdgcn_sched_barrier(0);
      const int l = 2 * (tid() + u * kResThreads);
      const double2 po = *reinterpret_cast<const double2*>(lds.p + l);
      const double2 d = q.diag(u);
      if (wide) {
        // |dx| / |x|, and |dx| where x = 0, of dx = rs alpha p^ and x = rs x^, rs = d^-1/2 (in
        // a branch of its own: computed for every cell the root cost an iteration 3 to 5 %)
        double x0 = fabs(q.x[u][0]), x1 = fabs(q.x[u][1]);
        if ((!(x0 > 0.0) && po.x != 0.0) || (!(x1 > 0.0) && po.y != 0.0)) {
          if (!(x0 > 0.0)) x0 = sqrt(d.x);
          if (!(x1 > 0.0)) x1 = sqrt(d.y);
        }
        linf = fmax(linf, fmax(fabs(alpha * po.x) / x0, fabs(alpha * po.y) / x1));
      }
      q.x[u][0] = fma(alpha, po.x, q.x[u][0]);
      q.x[u][1] = fma(alpha, po.y, q.x[u][1]);
      q.r[u][0] = fma(-alpha, q.s[u][0], q.r[u][0]);
      q.r[u][1] = fma(-alpha, q.s[u][1], q.r[u][1]);
      double2 pn;
      pn.x = fma(beta, po.x, q.r[u][0]);
      pn.y = fma(beta, po.y, q.r[u][1]);
      *reinterpret_cast<double2*>(lds.p + l) = pn;
      const double a0 = q.r[u][0] * q.r[u][0], a1 = q.r[u][1] * q.r[u][1];
      rr += a0 + a1;
      rrd = fma(a0, d.x, fma(a1, d.y, rrd));
    }
    for (int h = 2 * tid(); h < nh; h += 2 * kResThreads) {
      const double2 sn = *reinterpret_cast<const double2*>(lds.ex + h);
      double2 rn = *reinterpret_cast<const double2*>(lds.rh + h), pn = *reinterpret_cast<const double2*>(lds.p + kCap + h);
      rn.x = fma(-alpha, sn.x, rn.x);
      rn.y = fma(-alpha, sn.y, rn.y);
      pn.x = fma(beta, pn.x, rn.x);
      pn.y = fma(beta, pn.y, rn.y);
      *reinterpret_cast<double2*>(lds.rh + h) = rn;
      *reinterpret_cast<double2*>(lds.p + kCap + h) = pn;
    }
    __syncthreads();
  }
}

// Whether a refined solve has ended with an earlier launch.
__device__ __forceinline__ bool settled(const PcgScalars& o, const ResArgs& A) {
  return o.converged || o.nonfinite || o.inner_total >= A.max_iter || o.iter >= A.max_outer;
}

// The solve of one share of one problem.  false: a wait timed out.
template <int NP, ResMode kMode>
__device__ __forceinline__ bool solve_part(int my_part, unsigned char* dyn, Shared& S) {
  constexpr int kCap = 2 * NP * kResThreads;
  KernelArgs args = kernel_args();
  const DevLevel& L = args.L;
  const ResPlanDev& R = args.R;
  const ResArgs& A = args.A;
  my_part = __builtin_amdgcn_readfirstlane(my_part);
  ResPart me;  // (alike in every lane, which the compiler does not see of loaded values)
#pragma unroll
  for (int k = 0; k < int(sizeof(ResPart) / sizeof(int)); ++k)
    reinterpret_cast<int*>(&me)[k] = __builtin_amdgcn_readfirstlane(reinterpret_cast<const int*>(R.parts + my_part)[k]);
  const int ns = me.n_slots, n = L.n_slots;
  const int nh = 4 * me.n_units;
  double* const dl = reinterpret_cast<double*>(dyn);
  const ResLds at_lds(kCap, size_t(me.n_units), kMode == kCoupled ? size_t(me.n_coarse) : 0, kMode != kStreamed);
  Lds lds;
  lds.p = dl + at_lds.p;
  lds.rh = dl + at_lds.rh;
  lds.ex = dl + at_lds.ex;
  lds.partner = reinterpret_cast<int*>(dl + at_lds.partner);
  // nothing left to do: decided by an earlier launch, alike for every share
  if (A.resume && settled(A.sc[me.prob], A)) return true;
  const unsigned epoch0 = R.epoch[me.prob];
  Exchange X{R, me, my_part, epoch0, 0u, false};
  for (int u = tid(); u < me.n_units; u += kResThreads) lds.partner[u] = R.partner[me.unit0 + u];
  if (threadIdx.x == 0) {
    S.failed = int(R.epoch[2 * R.n_prob]);  // (looked at where the first exchange ends)
    if (my_part == me.part0) A.sc[me.prob].done = 0;  // set again when the whole record is written
  }
  auto take_halo = [&](double* dst) {  // the received values as the halo part of a vector
    for (int h = tid(); h < 4 * me.n_units; h += kResThreads) dst[h] = lds.ex[h];
  };

  // start: rs = diag^-1/2 exchanged, the scaled operator; x^_0 = x_0 / rs exchanged,
  // r^_0 = rs b - A^ x^_0 exchanged.  Every array is read once, in order; a thread's pairs
  // past the share's end read its first pair and get rs = 0, hence a zero operator.
  Regs<NP, kMode> q;
  q.face = 0;
  if constexpr (kMode == kStreamed)
    q.cs = reinterpret_cast<double2*>(static_cast<double*>(R.extra) + size_t(blockIdx.x) * kResStreamDoubles);
  else q.d = dl + at_lds.diag;
  if constexpr (kMode == kCoupled) {
    q.cv = dl + at_lds.coarse;
    q.uc0 = 4 * (me.n_units - me.n_coarse);
  }
  double v[kSums] = {0.0, 0.0, 0.0, 0.0}, m = -DBL_MAX;
  auto slot = [&](int l) -> int64_t { return me.slot0 + (l < ns ? l : 0); };
  auto pair = [&](const double* a, int64_t i) { return *reinterpret_cast<const double2*>(a + i); };
  auto at = [&](int l) { return *reinterpret_cast<const double2*>(lds.p + l); };
  {
    double2 d[NP];
    uint2 pl[NP];
#pragma unroll
    for (int u = 0; u < NP; ++u) {
      const int64_t i = slot(2 * (tid() + u * kResThreads));
      d[u] = pair(A.diag, i);
      pl[u] = R.places[i >> 1];
    }
#pragma unroll
    for (int u = 0; u < NP; ++u) {
      const int l = 2 * (tid() + u * kResThreads);
      const bool valid = l < ns;
      const double2 rs{valid ? 1.0 / sqrt(d[u].x) : 0.0, valid ? 1.0 / sqrt(d[u].y) : 0.0};
      m = fmax(m, fmax(-d[u].x, -d[u].y));
      q.put_diag(u, d[u]);
      *reinterpret_cast<double2*>(lds.p + l) = rs;
      auto place = [&](unsigned c, unsigned own) {
        if (!valid) return own;
        return (c & kResHalo) ? unsigned(kCap) + (c & ~kResHalo) : c;
      };
      const unsigned x0 = place(pl[u].x & 0xffffu, l), x1 = place(pl[u].x >> 16, l + 1);
      const unsigned y = place(pl[u].y & 0xffffu, l), z = place(pl[u].y >> 16, l);
      q.px[u] = x0 | (x1 << 16);
      q.pyz[u] = y | (z << 16);
      if (max(max(x0, x1), max(y, z)) >= unsigned(kCap)) q.face |= 1u << u;
      if constexpr (kMode == kCoupled) {
        q.cu[u] = valid ? static_cast<const unsigned*>(R.extra)[(me.slot0 + l) >> 1] : 0u;
        keep(q.cu[u]);
      }
      keep(q.px[u]);
      keep(q.pyz[u]);
      stage(q, lds.ex, u, rs.x, rs.y);
    }
  }
  __syncthreads();
  if (!exchange(X, A.meet_limit, v, m, true, S, lds)) return false;
  const double dmin = -m;
  take_halo(lds.p + kCap);
  // from here on units between shares on the same XCD go through its L2
  for (int u = tid(); u < me.n_units; u += kResThreads) {
    const int2 peer = reinterpret_cast<const int2*>(R.partner + R.far_units())[me.unit0 + u];
    if (S.xcc[peer.y] == (unsigned char)xcc_id()) lds.partner[u] = R.far_units() + peer.x;
  }
  // (more than one XCD's compute units are needed where shares are larger)
  if constexpr (NP <= 2)
    if (R.n_prob == 1 && me.group > 1)
      X.one_xcd = __builtin_amdgcn_readfirstlane(
                      __syncthreads_and(tid() >= me.group || S.xcc[tid()] == (unsigned char)xcc_id())) != 0;
  for (int k = 0; k < 32 && nh > 0 && k * kResThreads < 2 * nh + 8 * kResThreads; ++k) {
    const int unit = min(tid() + k * kResThreads, 2 * nh - 1) >> 3;  // (the last word's past the end, as it is read there)
    const int2 peer = reinterpret_cast<const int2*>(R.partner + R.far_units())[me.unit0 + unit];
    if (S.xcc[peer.y] == (unsigned char)xcc_id()) X.near |= 1u << k;
  }
  __syncthreads();
  if constexpr (kMode == kCoupled) {
    for (int k = tid(); k < 4 * me.n_coarse; k += kResThreads) {
      const int2 c = reinterpret_cast<const int2*>(static_cast<const unsigned*>(R.extra) + n / 2)[me.unit0 + me.n_units - me.n_coarse + (k >> 2)];
      const int d = c.y & 7, a = d >> 1, t0 = a == 0 ? 1 : 0, t1 = a == 2 ? 1 : 2;
      const int f = (c.y & ~7) | ((d & 1) << a) | ((k & 1) << t0) | (((k >> 1) & 1) << t1);
      q.cv[k] = L.cif[size_t(a) * n + f] * (lds.p[c.x] * lds.p[kCap + q.uc0 + k]);
    }
    __syncthreads();
  }
  // (one axis after the other, so that the loads in flight are few registers)
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    double2 cp[NP], cm[NP];
#pragma unroll
    for (int u = 0; u < NP; ++u) {
      const int64_t i = int64_t(a) * n + slot(2 * (tid() + u * kResThreads));
      cp[u] = pair(A.Cp, i);
      cm[u] = pair(A.Cm, i);
    }
#pragma unroll
    for (int u = 0; u < NP; ++u) {
      const int tt = tid(), l = 2 * (tt + u * kResThreads);
      const double2 rs = at(l);
      if (a == 0) {
        q.put_axis(u, 0, cp[u].x * (rs.x * rs.y), 0.0, cm[u].x * (rs.x * lds.p[q.px[u] & 0xffffu]),
                   cp[u].y * (rs.y * lds.p[q.px[u] >> 16]));
        continue;
      }
      const bool up = tt & a;  // on the + side of its oct
      const double2 in = up ? cm[u] : cp[u], out = up ? cp[u] : cm[u];
      const double2 rn = at(a == 1 ? q.pyz[u] & 0xffffu : q.pyz[u] >> 16);
      const double sx = a == 1 ? dpp<kQuadXor1>(rs.x, rs.x) : dpp<kQuadXor2>(rs.x, rs.x);
      const double sy = a == 1 ? dpp<kQuadXor1>(rs.y, rs.y) : dpp<kQuadXor2>(rs.y, rs.y);
      q.put_axis(u, a, in.x * (rs.x * sx), in.y * (rs.y * sy), out.x * (rs.x * rn.x), out.y * (rs.y * rn.y));
    }
  }
  {
    double2 x0[NP];
#pragma unroll
    for (int u = 0; u < NP; ++u) x0[u] = pair(A.x, slot(2 * (tid() + u * kResThreads)));
#pragma unroll
    for (int u = 0; u < NP; ++u) {
      const int l = 2 * (tid() + u * kResThreads);
      const double2 rs = at(l);
      q.s[u][0] = rs.x;
      q.s[u][1] = rs.y;
      q.x[u][0] = l < ns ? x0[u].x / rs.x : 0.0;
      q.x[u][1] = l < ns ? x0[u].y / rs.y : 0.0;
      keep(q.x[u][0]);
      keep(q.x[u][1]);
      stage(q, lds.ex, u, q.x[u][0], q.x[u][1]);
    }
  }
  v[0] = v[1] = v[2] = v[3] = 0.0;
  __syncthreads();  // rs read everywhere
#pragma unroll
  for (int u = 0; u < NP; ++u)
    *reinterpret_cast<double2*>(lds.p + 2 * (tid() + u * kResThreads)) = double2{q.x[u][0], q.x[u][1]};
  if (!exchange(X, A.spin_limit, v, m, false, S, lds)) return false;
  take_halo(lds.p + kCap);
  __syncthreads();
  v[0] = v[1] = v[2] = v[3] = 0.0;
  {
    double2 b[NP];
    int2 ch[NP];
#pragma unroll
    for (int u = 0; u < NP; ++u) {
      const int64_t i = slot(2 * (tid() + u * kResThreads));
      b[u] = pair(A.b, i);
      ch[u] = *reinterpret_cast<const int2*>(L.child + i);
    }
    apply_all(q, lds.p, [&](int u, const double(&)[2], const double(&av)[2]) {
      const int l = 2 * (tid() + u * kResThreads);
      const double2 d = q.diag(u);
      q.r[u][0] = q.s[u][0] * b[u].x - av[0];
      q.r[u][1] = q.s[u][1] * b[u].y - av[1];
      keep(q.r[u][0]);
      keep(q.r[u][1]);
      v[0] += (q.r[u][0] * d.x) * q.r[u][0] + (q.r[u][1] * d.y) * q.r[u][1];
      if (l < ns && ch[u].x == -1) v[1] += b[u].x * b[u].x;
      if (l < ns && ch[u].y == -1) v[1] += b[u].y * b[u].y;
      stage(q, lds.ex, u, q.r[u][0], q.r[u][1]);
    });
  }
  __syncthreads();  // x^ read everywhere
#pragma unroll
  for (int u = 0; u < NP; ++u)
    *reinterpret_cast<double2*>(lds.p + 2 * (tid() + u * kResThreads)) = double2{q.r[u][0], q.r[u][1]};
  if (!exchange(X, A.spin_limit, v, m, false, S, lds)) return false;
  take_halo(lds.rh);
  take_halo(lds.p + kCap);
  __syncthreads();
  // (a resumed solve keeps the norms and the threshold of its first launch)
  const double start2 = v[0];
  const double rnorm0 = A.resume ? A.sc[me.prob].rnorm0 : sqrt(v[0]), bnorm = sqrt(v[1]);
  const double floor_b = A.abs_floor * bnorm, thresh = A.resume ? A.sc[me.prob].thresh : fmax(A.tol * rnorm0, floor_b);
  const int before = A.resume ? A.sc[me.prob].inner_total : 0;
  const int outer = __builtin_amdgcn_readfirstlane(A.resume ? A.sc[me.prob].iter : 0);
  CgResult res;
  res.rn = sqrt(start2);
  res.linf = 0.0;
  res.iters = res.segments = 0;
  res.fin = isfinite(start2) && isfinite(bnorm);
  res.conv = res.fin && res.rn <= floor_b;
  const long long clk0 = wall_clock64();
  S.gate[tid() >> 6] = A.refine ? A.inner_tol * A.inner_tol * start2 : 1.000001 * thresh * thresh;
  if (res.fin && !res.conv &&
      !cg_loop(X, q, lds, S, thresh, A.tol, A.max_iter - before, A.linf_test != 0, dmin, A, A.max_outer - outer, res))
    return false;
  const long long clk1 = wall_clock64();
  args = kernel_args();

  // the unscaled iterate, the T update of the coupling term (linearised emission), the
  // true residual b - (A^ x^) / rs and the smallest leaf energy
  v[0] = v[1] = v[2] = v[3] = 0.0;
  m = -DBL_MAX;
  if (threadIdx.x == 0) st_word32(R.epoch + R.n_prob + me.prob, epoch0);
#pragma unroll
  for (int u = 0; u < NP; ++u) {
    __builtin_amdgcn_sched_barrier(0);
    const int l = 2 * (tid() + u * kResThreads);
    if (l < ns) {
      const int64_t i = me.slot0 + l;
      const double2 d = q.diag(u);
      const double rs[2] = {1.0 / sqrt(d.x), 1.0 / sqrt(d.y)};
      double2 xi{q.x[u][0] * rs[0], q.x[u][1] * rs[1]};
      if (res.iters > 0) *reinterpret_cast<double2*>(A.x + i) = xi;
      else xi = pair(A.x, i);
      const int2 ch = *reinterpret_cast<const int2*>(L.child + i);
      if (ch.x == -1) m = fmax(m, -xi.x);
      if (ch.y == -1) m = fmax(m, -xi.y);
      if (A.cp.T) {
#pragma unroll 1
        for (int e = 0; e < 2; ++e)
          if ((e ? ch.y : ch.x) == -1) {
            const double T = A.cp.T[i + e], rr = A.rho[i + e], xe = e ? xi.y : xi.x;
            const double eta = A.cp.kappa_P * rr * A.cp.c_light * A.dt;
            const double bT = 4.0 * A.cp.a_rad * T * T * T;
            A.T_out[i + e] = T + eta * (xe - A.cp.a_rad * (T * T * T * T)) / (rr * A.cp.c_v + eta * bT);
          }
      }
      q.x[u][0] = xi.x / rs[0];
      q.x[u][1] = xi.y / rs[1];
    }
    if (A.true_residual) {
      *reinterpret_cast<double2*>(lds.p + l) = double2{q.x[u][0], q.x[u][1]};
      stage(q, lds.ex, u, q.x[u][0], q.x[u][1]);
    }
  }
  if (A.true_residual) {
    double none = 0.0;
    __syncthreads();
    if (!exchange(X, A.spin_limit, v, none, false, S, lds)) return false;
    take_halo(lds.p + kCap);
    __syncthreads();
    v[0] = v[1] = v[2] = v[3] = 0.0;
    apply_all(q, lds.p, [&](int u, const double(&)[2], const double(&av)[2]) {
      const int l = 2 * (tid() + u * kResThreads);
      if (l < ns) {
        const double2 b = *reinterpret_cast<const double2*>(A.b + me.slot0 + l);
        const double2 d = q.diag(u);
        const double r0 = b.x - av[0] * sqrt(d.x), r1 = b.y - av[1] * sqrt(d.y);
        v[0] = fma(r0, r0, fma(r1, r1, v[0]));
      }
    });
  }
  v[1] = v[2] = v[3] = 0.0;
  put_sums(X, v, m, true, S, static_cast<const double*>(nullptr), lds.partner);
  if (my_part != me.part0) return true;
  if (!collect(X, A.spin_limit, v, m, true, S, static_cast<double*>(nullptr))) return false;
  if (threadIdx.x == 0) {
    R.epoch[me.prob] = X.epoch;
    PcgScalars z{};
    if (A.refine && res.iters > 0) {
      // the stop is decided on the true residual; a start at the floor needed no sweep
      res.rn = sqrt(v[0]);
      res.fin = res.fin && isfinite(res.rn);
      res.conv = res.fin && ((res.rn <= thresh && (!A.linf_test || res.linf < A.tol)) || res.rn == 0.0);
    }
    z.rnorm0 = rnorm0;
    z.bnorm = bnorm;
    z.thresh = thresh;
    z.tol = A.tol;
    z.abs_floor = A.abs_floor;
    z.rnorm = res.rn;
    z.linf = res.linf;
    z.true_rnorm = sqrt(v[0]);
    z.min_E = -m;
    z.iter = A.refine ? outer + res.segments : res.iters;
    z.inner_total = A.refine ? before + res.iters : 0;
    z.done = 1;
    z.converged = res.conv ? 1 : 0;
    z.nonfinite = res.fin ? 0 : 1;
    z.max_iter = A.max_iter;
    z.linf_test = A.linf_test;
    // the constant 100 MHz counter; of all launches of a refined solve
    z.loop_ms = (A.resume ? A.sc[me.prob].loop_ms : 0.0) + double(clk1 - clk0) * 1e-5;
    A.sc[me.prob] = z;
  }
  return true;
}

// The tasks of a block, [first, end), and the share of one.
struct Tasks {
  int first, end;
};
__device__ __forceinline__ Tasks tasks_of_block(const KernelArgs& k) {
  const int b = int(blockIdx.x);
  if (k.A.spread) return Tasks{b, b + 1};
  return Tasks{k.R.task0[b], k.R.task0[b + 1]};
}
__device__ __forceinline__ int share_of(const KernelArgs& k, int task) { return k.A.spread ? task : k.R.task[task]; }

// A block that gave up at a task leaves: none of the problems it leads from there on is
// completed by this launch.
__device__ __forceinline__ void give_up(int task) {
  if (threadIdx.x != 0) return;
  const KernelArgs args = kernel_args();
  const ResPlanDev& R = args.R;
  const ResArgs& A = args.A;
  st_word32(R.epoch + 2 * R.n_prob, 1u);
  for (const int end = tasks_of_block(args).end; task < end; ++task) {
    const int part = share_of(args, task);
    const ResPart& p = R.parts[part];
    PcgScalars& o = A.sc[p.prob];
    if (part == p.part0 && !(A.resume && settled(o, A))) o.done = 0;
  }
}

template <int NP, ResMode kMode>
__global__ __launch_bounds__(kResThreads) void k_cg_resident(KernelArgs) {
  extern __shared__ __align__(16) unsigned char res_lds[];
  __shared__ Shared S;
  const Tasks t = tasks_of_block(kernel_args());
  for (int k = t.first; k < t.end; ++k) {
    if (!solve_part<NP, kMode>(share_of(kernel_args(), k), res_lds, S)) {
      give_up(k);
      return;
    }
    __syncthreads();
  }
}

// Shares of several sizes in one launch: each runs with as many pairs per thread as it
// needs (a small share in the loops of a large one would mostly iterate over nothing).
__global__ __launch_bounds__(kResThreads) void k_cg_resident_batch(KernelArgs) {
  extern __shared__ __align__(16) unsigned char res_lds[];
  __shared__ Shared S;
  const Tasks t = tasks_of_block(kernel_args());
  for (int k = t.first; k < t.end; ++k) {
    const KernelArgs now = kernel_args();
    const int part = share_of(now, k);
    bool ok;
    switch ((now.R.parts[part].n_slots + 2 * kResThreads - 1) / (2 * kResThreads)) {
      case 1: ok = solve_part<1, kHeld>(part, res_lds, S); break;
      case 2: ok = solve_part<2, kHeld>(part, res_lds, S); break;
      case 3: ok = solve_part<3, kHeld>(part, res_lds, S); break;
      case 4: ok = solve_part<4, kHeld>(part, res_lds, S); break;
      case 5: ok = solve_part<5, kHeld>(part, res_lds, S); break;
      case 6: ok = solve_part<6, kStreamed>(part, res_lds, S); break;
      default: ok = solve_part<8, kStreamed>(part, res_lds, S);
    }
    if (!ok) {
      give_up(k);
      return;
    }
    __syncthreads();
  }
}

// What a launch may ask for beside Shared and the 256 bytes of __syncthreads_and.  (That
// much is a function's default: its attribute is left alone, which all threads share.)
constexpr size_t kLdsLimit = 160 * 1024 - ((sizeof(Shared) + 15) & ~size_t(15)) - 256;

// Pairs of slots per thread of a share (a batch has no loops of 7: see its kernel).
int pairs_of(int n_slots, int n_prob) {
  const int np = (n_slots + 2 * kResThreads - 1) / (2 * kResThreads);
  return n_prob > 1 && np == 7 ? 8 : np;
}

hipError_t launch_kernel(void (*f)(KernelArgs), hipStream_t s, const DevLevel& L, const ResPlanDev& R,
                         const ResArgs& A) {
  hipLaunchKernelGGL(f, dim3(A.spread ? R.n_parts : R.n_blocks), dim3(kResThreads), R.lds, s, KernelArgs{L, R, A});
  return hipGetLastError();
}

}  // namespace

// The shares of one problem run with as many pairs as its largest.
int resident_lds(const std::vector<ResPart>& parts, int max_slots, int n_prob) {
  size_t most = 0;
  for (const ResPart& p : parts) {
    const int np = pairs_of(n_prob > 1 ? p.n_slots : max_slots, n_prob);
    most = std::max(most, ResLds(2 * size_t(np) * kResThreads, p.n_units, p.n_coarse, np <= kResPairs).bytes);
  }
  return int(std::min<size_t>(most, 1u << 30));
}

size_t resident_coefs(const ResPlanDev& R) {
  return R.max_slots > kResBlockSlots ? size_t(R.n_blocks) * kResStreamDoubles : 0;
}

bool resident_fits(const ResPlanDev& R) {
  return R.n_parts > 0 && R.max_slots <= kResMaxSlots && size_t(R.lds) <= kLdsLimit;
}

hipError_t launch_resident(hipStream_t s, const DevLevel& L, const ResPlanDev& R, const ResArgs& A) {
  if (R.n_prob > 1) return launch_kernel(&k_cg_resident_batch, s, L, R, A);
  if (R.coupled) {
    switch (pairs_of(R.max_slots, 1)) {
      case 1: return launch_kernel(&k_cg_resident<1, kCoupled>, s, L, R, A);
      case 2: return launch_kernel(&k_cg_resident<2, kCoupled>, s, L, R, A);
      case 3: return launch_kernel(&k_cg_resident<3, kCoupled>, s, L, R, A);
      case 4: return launch_kernel(&k_cg_resident<4, kCoupled>, s, L, R, A);
      case 5: return launch_kernel(&k_cg_resident<5, kCoupled>, s, L, R, A);
    }
    return hipErrorNotSupported;
  }
  switch (pairs_of(R.max_slots, 1)) {
    case 1: return launch_kernel(&k_cg_resident<1, kHeld>, s, L, R, A);
    case 2: return launch_kernel(&k_cg_resident<2, kHeld>, s, L, R, A);
    case 3: return launch_kernel(&k_cg_resident<3, kHeld>, s, L, R, A);
    case 4: return launch_kernel(&k_cg_resident<4, kHeld>, s, L, R, A);
    case 5: return launch_kernel(&k_cg_resident<5, kHeld>, s, L, R, A);
    case 6: return launch_kernel(&k_cg_resident<6, kStreamed>, s, L, R, A);
    case 7: return launch_kernel(&k_cg_resident<7, kStreamed>, s, L, R, A);
    case 8: return launch_kernel(&k_cg_resident<8, kStreamed>, s, L, R, A);
  }
  return hipErrorNotSupported;
}

}  // namespace amrfld
