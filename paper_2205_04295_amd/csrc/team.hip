// The M-rPIE sweep as one persistent launch (Methods, "M-rPIE algorithm",
// Eq. 4-7): a reconstruction is run from its first position to its last by a
// team of workgroups that sit on one XCD.
//
// Why one XCD.  The 2-D FFT of a position exchanges all spectra between its
// row and its column transforms twice.  Workgroups on different XCDs can only
// exchange through memory: data written by one kernel and read on another XCD
// by the next comes at about 3 TB/s for the whole chip, and a barrier over
// all XCDs costs 3.8 us (launch boundaries about 2 us each).  On one XCD the
// exchange stays in its 4 MB L2 (reads at more than four times that rate) and
// a barrier of 32 workgroups costs well under 1 us, so a position is three
// phases with a team barrier after each:
//
//   gather   rows of the box: exit waves (Eq. 1, 4), forward row FFTs
//   columns  forward column FFTs, modulus (Eq. 7), inverse column FFTs
//   update   inverse row FFTs, probe rows (Eq. 5), object rows (Eq. 6)
//
// The 8 XCDs run 8 teams side by side (more and smaller ones for small
// probes) and pull jobs from a queue, so a batch needs no lock step and no
// launch per position.
//
// Who does what.  A unit is G = 64 / L adjacent rows (in the columns phase:
// columns) of the box, one wave's worth of transforms of one mode (wfft.hpp:
// every FFT runs inside a wave, so waves wait for each other only where data
// is exchanged).  The modes of a unit go to different waves of one workgroup
// (KM of them to each wave), which add up what Eq. 6 and Eq. 7 sum over the
// modes through the LDS, so one wave's loads, LDS exchanges and stores hide
// behind the others' arithmetic: one wave per SIMD that took a unit's three
// modes in turn needed 15.3 us a position of 256^2 x 3 where three waves per
// SIMD (WV = 12, which leaves 168 registers a lane) take 13.8; other mode
// counts have no use for 12 waves and run 8 with 248 registers.  A wave keeps
// its rows of the probe in registers for the whole job, and its box rows from
// the gather to the update: 3 of the 8 passes over a spectrum-sized array
// less, and the probe out of the L2, which at 256^2 x 3 it would fill up.
//
// Coherence.  All members of a team read the same XCC id, so they share one
// L2: a store is visible to the team once it is acknowledged (vmcnt 0 before
// the barrier), and loads of data that other members write carry sc1 (relaxed
// agent-scope atomics), which bypasses the CU's L1.  Agent fences, which
// would walk the L2 (8 us each), are not needed inside a team; jobs share no
// written memory, and the kernel's end publishes everything.
//
// No wait depends on a workgroup that may not have started: a team is formed
// of the workgroups that have arrived when its leader closes the list (all of
// them as a rule; the leader waits up to 10 ms for stragglers), later ones
// leave at once.  A team that came out too small for its job's units runs the
// job in loops over them (run_loops), slowly but to the same bits.
#include <algorithm>
#include <mutex>
#include <vector>

#include "sweep.hpp"
#include "wfft.hpp"

namespace mrpie {
namespace {

constexpr int kMaxWaves = 12;     // of a workgroup (template parameter WV: 8 or 12)
constexpr int kMaxXcc = 16;       // values the XCC id register can take
constexpr int kMaxSize = kTeamMembers;  // members of a team
// Jobs are of four classes by the members they need: teams of 32, 16, 8, 4.
// The workgroups of an XCD take the jobs of class 0 as one team, then those
// of class 1 as two teams, and so on.
constexpr int kClasses = 4;
constexpr int kMaxTeams = 15;     // teams of an XCD over all classes: 1 + 2 + 4 + 8
constexpr int kMaxTeamJobs = 384; // jobs of one launch (pointers in the kernel arguments)
constexpr int kSide = 2;          // transforms of a lane group side by side
constexpr long long kMaxPositions = 1024;   // of a team in one launch (6 to 15 us each)
constexpr unsigned kClosed = 0x40000000u;
constexpr long long kFormTicks = 1000000;      // 10 ms of the 100 MHz wall clock
constexpr int kSpinTicks = 2000000000;         // 20 s: a wait inside a job that ends so late is an error
constexpr long long kIdleTicks = 1000000000000LL;  // ... of members without work, for the others' job

// One job as the teams read it, in the job's own workspace (psi[1], which the
// team sweep does not use otherwise), behind the control words of the launch
// (in the first job's).
struct TeamJob {
  JobRec j;
  float* err_out;
  Common c;
  int km;  // modes of a wave
};
constexpr size_t kCtrlBytes = 6144;
constexpr size_t kJobOffset = kCtrlBytes;  // of TeamJob inside psi[1]
// Behind it: for each of a position's three barriers and each member, the
// barriers passed and a value that travels with them.
constexpr size_t kFlagOffset = kJobOffset + 256;
constexpr int kFlagWords = 3 * kMaxSize * 2;
// control words: job queue heads, then per XCD 64 words: the arrival count,
// the closed count, then for team k, on 8 bytes, the arrivals at its barrier
// between jobs and the arrivals at which all members leave (0: not yet), and
// the job it runs
constexpr int kCtrlXcc = 64;
constexpr int kXccWords = 64;
static_assert((kCtrlXcc + kMaxXcc * kXccWords) * 4 <= kCtrlBytes && 2 + 4 * kMaxTeams <= kXccWords, "control words");
static_assert(sizeof(TeamJob) <= 256 && kFlagOffset + kFlagWords * 4 <= 8192, "psi[1] of 32^2 x 1");

struct TeamArgs {
  unsigned* ctrl;
  int expect;                    // workgroups of each XCD
  int limit;                     // ... of which teams are formed at most
  int spin;                      // ticks after which a wait inside a job gives up
  int nxcc, from, xccs;          // XCDs of the device, the first of the launch and how many of them
  int first[kClasses + 1];       // job[first[c] .. first[c + 1]) are class c's, longest first
  const TeamJob* job[kMaxTeamJobs];
};
static_assert(sizeof(TeamArgs) <= 4096, "kernel arguments");

#define MRPIE_AS1 __attribute__((address_space(1)))
#define MRPIE_AS4 __attribute__((address_space(4)))

__device__ __forceinline__ unsigned ld_agent(const unsigned* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_agent(unsigned* p, unsigned v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned add_agent(unsigned* p, unsigned v) {
  return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Global memory by address: a job's pointers are read from memory, where the
// compiler cannot tell their address space and would use flat instructions,
// whose waits are also LDS waits.  `at` adds a 32-bit byte offset of the
// lane, so that the address is a scalar base plus one register.
struct Glob {
  MRPIE_AS1 char* p;
  __device__ __forceinline__ Glob() {}
  __device__ __forceinline__ explicit Glob(const void* q) : p((MRPIE_AS1 char*)(void*)q) {}
  __device__ __forceinline__ Glob at(unsigned bytes) const {
    Glob g;
    g.p = p + bytes;
    return g;
  }
  __device__ __forceinline__ Glob far(size_t bytes) const {
    Glob g;
    g.p = p + bytes;
    return g;
  }
  template <typename T>
  __device__ __forceinline__ T ld() const {
    return *(const MRPIE_AS1 T*)p;
  }
  template <typename T>
  __device__ __forceinline__ void st(T v) const {
    *(MRPIE_AS1 T*)p = v;
  }
  // values that another member of the team may have written: sc1, past the L1
  template <typename T>
  __device__ __forceinline__ T ld_team() const {
    return __hip_atomic_load((const MRPIE_AS1 T*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ __forceinline__ float2 ld2() const {
    typedef float v2 __attribute__((ext_vector_type(2)));
    const v2 v = ld<v2>();
    return mk(v.x, v.y);
  }
  __device__ __forceinline__ float2 ld2_team() const {
    const unsigned long long v = ld_team<unsigned long long>();
    return mk(__uint_as_float((unsigned)v), __uint_as_float((unsigned)(v >> 32)));
  }
  __device__ __forceinline__ void st2(float2 v) const {
    typedef float v2 __attribute__((ext_vector_type(2)));
    st<v2>(v2{v.x, v.y});
  }
};

// The arithmetic of a position, with its fused operations spelled out and no
// others: run_units and run_loops compute the same bits, and left to itself
// the compiler fuses a product into a sum or not by what stands around it
// (the FFTs' sums are fused the same everywhere: nothing here fuses into them).
#pragma clang fp contract(off)
__device__ __forceinline__ float2 xmul(float2 a, float2 b) {  // a b
  return mk(fmaf(a.x, b.x, -(a.y * b.y)), fmaf(a.x, b.y, a.y * b.x));
}
__device__ __forceinline__ float2 xmulc(float2 a, float2 b) {  // a conj(b)
  return mk(fmaf(a.x, b.x, a.y * b.y), fmaf(a.y, b.x, -(a.x * b.y)));
}
__device__ __forceinline__ float2 xnmac(float2 v, float2 a, float2 b) {  // v - a b
  return mk(fmaf(a.y, b.y, fmaf(-a.x, b.x, v.x)), fmaf(-a.y, b.x, fmaf(-a.x, b.y, v.y)));
}
__device__ __forceinline__ float2 xaxpy(float2 v, float2 a, float s) {  // v + s a
  return mk(fmaf(a.x, s, v.x), fmaf(a.y, s, v.y));
}
__device__ __forceinline__ float2 xscale(float2 a, float s) { return mk(a.x * s, a.y * s); }
__device__ __forceinline__ float xabs2(float2 a) { return fmaf(a.x, a.x, a.y * a.y); }
__device__ __forceinline__ float xadd_abs2(float s, float2 a) { return fmaf(a.x, a.x, fmaf(a.y, a.y, s)); }
__device__ __forceinline__ float xadd_dot(float s, float2 a, float2 b) {  // s + Re(a conj(b))
  return s + fmaf(a.x, b.x, a.y * b.y);
}
__device__ __forceinline__ float xadd_cross(float s, float2 a, float2 b) {  // s + Im(a conj(b))
  return s + fmaf(a.y, b.x, -(a.x * b.y));
}
// w top + (1 - w) v, the denominators of Eq. 5 and Eq. 6
__device__ __forceinline__ float xblend(float w, float top, float v) { return fmaf(1.f - w, v, w * top); }
// |Psi| - sqrt(I) at a pixel of power A, rs = 1 / sqrt(A), sq = sqrt(I)
__device__ __forceinline__ float xmisfit(float A, float rs, float invN, float sq) { return fmaf(A * rs, invN, -sq); }
#pragma clang fp contract(fast)

// HW_REG_XCC_ID: the XCD this workgroup runs on
__device__ __forceinline__ int xcc_id() { return __builtin_amdgcn_s_getreg((3 << 11) | 20) & (kMaxXcc - 1); }

// The members of a team as one of them sees it.
struct Team {
  int rank, size;
  unsigned* bar;     // arrivals, counted up; behind it when to leave, and the job being run
  unsigned target;   // arrivals that end the next barrier
};

// p += 1 by one lane of the wave.  The lane is chosen inside the asm block,
// not by a divergent branch: register copies that the compiler places at the
// join of such a branch have landed before the restore of exec, where the
// other lanes lose them.  The phases below have no divergent branch for the
// same reason: one-lane stores are stores of one value by all lanes.
__device__ __forceinline__ void add_one(unsigned* p) {
  unsigned long long exec;
  asm volatile(
      "s_mov_b64 %0, exec\n"
      "s_mov_b64 exec, 1\n"
      "global_atomic_add %1, %2, %3\n"
      "s_mov_b64 exec, %0"
      : "=&s"(exec)
      : "v"(0), "v"(1), "s"(p)
      : "memory");
}
// p's value, the same for all lanes
__device__ __forceinline__ unsigned ld_uniform(const unsigned* p) {
  return __builtin_amdgcn_readfirstlane(ld_agent(p));
}

// Values the waves of a workgroup share (static LDS).
struct Shared {
  float part[kMaxWaves];   // each wave's maximum
  float top;               // the team's
  int ok;                  // 0: a wait took too long, leave
  int spin;                // (TeamArgs)
  int team, rank, size;
};

// Barrier over the workgroups of a team between jobs.  False: leave.  A member
// whose wait inside a job gave up says so before it arrives at the barrier that
// ends the job, and by that barrier's number: a slower one may still be reading
// at the barrier before it, which all must pass.  So all leave at the same one
// and none waits for a member that has left.  (The bound of this wait is a last
// resort: those it waits for are running, and their own waits end.)
__device__ __forceinline__ bool team_barrier(Team& tm, Shared* sh) {
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  tm.target += (unsigned)tm.size;
  if (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) == 0) {
    add_one(tm.bar);
    const long long t0 = wall_clock64();
    for (;;) {
      const unsigned long long v = __hip_atomic_load((const unsigned long long*)tm.bar, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT);
      const unsigned here = __builtin_amdgcn_readfirstlane((unsigned)v);
      const unsigned leave = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
      if ((int)(here - tm.target) >= 0) {
        if (leave && (int)(tm.target - leave) >= 0) sh->ok = 0;
        break;
      }
      if (wall_clock64() - t0 > kIdleTicks) {
        st_agent(tm.bar + 1, tm.target);
        sh->ok = 0;
        break;
      }
      __builtin_amdgcn_s_sleep(2);
    }
  }
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(sh->ok) != 0;
}

// Barriers inside a job.  Barrier b (0, 1, 2: after the gather, the columns,
// the update) publishes every store of the members to the team and gives the
// largest of all sh->part.  Each member raises its own flag, the value beside
// it, and watches all of them in one load: no shared counter (0.75 us with
// one), and the maxima that Eq. 5 and Eq. 6 divide by need no memory pass of
// their own.  (A flag is raised again one position later; by then every
// member has passed another barrier and so has read it.)
template <int WV>
struct JobBarrier {
  Glob flags;
  int rank, size;
  Shared* sh;
  int spin;            // (TeamArgs)
  unsigned epoch = 0;  // positions begun
  __device__ __forceinline__ float operator()(int b) const {
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __syncthreads();
    if (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) == 0) {
      const int lane = threadIdx.x & 63;
      float top = wave_max(lane < WV ? sh->part[lane < WV ? lane : 0] : 0.f);
      if (size > 1) {
        const Glob fl = flags.far((size_t)b * (kMaxSize * 8));
        fl.far((size_t)rank * 8).st<unsigned long long>((unsigned long long)epoch |
                                                        (unsigned long long)__float_as_uint(top) << 32);
        asm volatile("" ::: "memory");
        const Glob one = fl.at((lane < size ? lane : 0) * 8);
        const long long t0 = wall_clock64();
        unsigned long long v;
        for (;;) {
          v = one.ld_team<unsigned long long>();
          if (__builtin_amdgcn_ballot_w64((int)((unsigned)v - epoch) >= 0) == ~0ull) break;
          if (wall_clock64() - t0 > spin) {
            sh->ok = 0;
            break;
          }
        }
        top = wave_max(__uint_as_float((unsigned)(v >> 32)));
      }
      sh->top = top;
    }
    __syncthreads();
    return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(sh->top)));
  }
  __device__ __forceinline__ bool ok() const { return __builtin_amdgcn_readfirstlane(sh->ok) != 0; }
};

// Where the two halves of a position's transforms meet: the spectra of a
// team's job in 4 x 4 tiles of one 128-byte line, so that a wave holding rows
// and a wave holding columns both touch whole lines (row-major: a column
// access takes 16 bytes of each line).
template <int N>
__device__ __forceinline__ unsigned tile_idx(unsigned k, unsigned c) {
  return (((k >> 2) * (N / 4) + (c >> 2)) << 4) | ((k & 3) << 2) | (c & 3);
}

// A lane's transform (group), its place in it, and the group's scratch.  The
// lane number is hidden from the compiler, so the index arithmetic of a phase
// stays in the phase instead of being hoisted out of the position loop, where
// hundreds of addresses would be live (and spill).
template <int N>
struct Lane {
  unsigned grp, l;
  float2* sc;
  __device__ __forceinline__ explicit Lane(float2* wave_scratch) {
    unsigned t = threadIdx.x & 63;
    asm volatile("" : "+v"(t));
    grp = t % WaveFft<N>::G;
    l = t / WaveFft<N>::G;
    sc = wave_scratch + grp * WaveFft<N>::PLEN;
  }
};

// Transforms P .. K - 1 of v, kSide of them side by side (by recursion: a loop
// this large is not unrolled, and v would be in memory).
template <typename F, int KM, int P, bool INV>
__device__ __forceinline__ void side_by_side(const F& f, float2 (*v)[F::PT], float2* sc, int l) {
  constexpr int K = KM - P < kSide ? KM - P : kSide;
  f.template run<K, INV>(v + P, sc, l);
  if constexpr (P + K < KM) side_by_side<F, KM, P + K, INV>(f, v, sc, l);
}

// How a job's units and modes are dealt to a team.
template <int N, int KM, int WV>
struct Deal {
  using F = WaveFft<N>;
  static constexpr int NU = N / F::G;  // units
  int M, MW, UW;                       // modes; waves of a unit; units of a workgroup
  __device__ __forceinline__ explicit Deal(int modes, int size) : M(modes), MW((modes + KM - 1) / KM) {
    UW = 1;
    while (UW * 2 * MW <= WV && UW * size < NU) UW *= 2;
  }
  __device__ __forceinline__ bool fits(int size) const { return MW <= WV && UW * size >= NU; }
  __device__ __forceinline__ int members() const { return (NU + UW - 1) / UW; }  // with units
};

// LDS of a workgroup: its pattern columns, the twiddles (if its transforms
// read them there), then per wave the scratch of its transforms and a plane of floats for the sums over modes (the whole of it
// for the three sums of the update, when no transform needs the scratch).
template <int N, int WV>
struct TeamLds {
  using F = WaveFft<N>;
  static constexpr int kFft = F::SCRATCH * 8;
  static constexpr int kSum = F::PT * 256;
  static constexpr int kWave = ((kFft + kSum > 3 * kSum ? kFft + kSum : 3 * kSum) + 15) & ~15;
  static constexpr int kPat = N * (8 * F::G < N ? 8 * F::G : N) * 4;  // of 8 units at most
  static constexpr int kHead = kPat + (F::kTable ? N * 8 : 0);
  static constexpr int kBytes = kHead + WV * kWave;
};

// The transforms' twiddles, in registers or (valid after the next barrier) at
// `tab` in the LDS.
template <int N>
__device__ __forceinline__ void init_fft(WaveFft<N>& f, float2* tab) {
  constexpr int ni = N == 64 ? 0 : N == 128 ? 1 : N == 192 ? 2 : N == 256 ? 3 : 4;
  if constexpr (WaveFft<N>::kTable) {
    const unsigned t = threadIdx.x < N ? threadIdx.x : N - 1;
    tab[t] = g_tw[ni][t];
    f.init(tab, 0);
  } else {
    f.init(g_tw[ni], (threadIdx.x & 63) / WaveFft<N>::G);
  }
}

// An iteration's error from its units' shares, in a fixed order (one wave).
template <int NU>
__device__ __forceinline__ void iteration_error(const Glob& gerr, const Glob& gis, float* err_out, int it) {
  const int lane = threadIdx.x & 63;
  double e = 0.0, v = 0.0;
#pragma unroll
  for (int i = 0; i < (NU + 63) / 64; ++i) {
    const unsigned q = lane + 64 * i;
    const size_t at = (size_t)it * kErrSlots * 8;
    const unsigned long long a = gerr.far(at).at((q < NU ? q : 0) * 8).ld_team<unsigned long long>();
    const unsigned long long b = gis.far(at).at((q < NU ? q : 0) * 8).ld_team<unsigned long long>();
    e += q < NU ? __longlong_as_double((long long)a) : 0.0;
    v += q < NU ? __longlong_as_double((long long)b) : 0.0;
  }
  e = wave_sum(e);
  v = wave_sum(v);
  Glob(err_out + it).st<float>((float)(v > 0.0 ? e / v : e));
}

// The whole sweep of one job by a team that has a wave for every unit and
// KM of its modes.
template <int N, int KM, int WV>
__device__ __forceinline__ void run_units(const Common& cm, const JobRec& jb, float* err_out, int rank, int size,
                                          char* lds, Shared* sh) {
  using F = WaveFft<N>;
  using D = Deal<N, KM, WV>;
  using S = TeamLds<N, WV>;
  constexpr int L = F::L, PT = F::PT, G = F::G, NU = D::NU;
  constexpr int GR = PT / 4;  // groups of four points, the unit in which sums are shared out
  constexpr unsigned NN = N * N;
  typedef float v4 __attribute__((ext_vector_type(4)));
  const int M = jb.M, J = jb.J, T = jb.T, H = jb.H, W = jb.W;
  const D deal(M, size);
  const int MW = deal.MW, UW = deal.UW;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ul = wave / MW, mw = KM > 1 && MW == 2 ? (wave ^ wave >> 2) & 1 : wave - ul * MW, u = rank * UW + ul;
  const bool active = ul < UW && u < NU;
  // Modes mw, mw + MW, ... of this wave.  Where M is no multiple of KM some
  // waves have one less; its registers hold zeros, which stay zeros.
  const int nk = KM == 1 ? 1 : (M - mw + MW - 1) / MW;
  const WsLayout ly = ws_layout(N, M, T);
  const Glob gobj(jb.obj), gprobe(jb.probe), gpos(jb.pos), gI(jb.I), ws(jb.ws);
  const Glob psi = ws.far(ly.psi[0]);
  const Glob gerr = ws.far(ly.err), gis = ws.far(ly.isum);
  const Glob flags = ws.far(ly.psi[1] + kFlagOffset);
  float* const s_pat = (float*)lds;
  char* const lds0 = lds;
  lds += S::kHead;
  char* const mine = lds + wave * S::kWave;

  F f;
  init_fft<N>(f, (float2*)(lds0 + TeamLds<N, WV>::kPat));

  JobBarrier<WV> barrier{flags, rank, size, sh, __builtin_amdgcn_readfirstlane(sh->spin)};
  // The spectra a wave holds as rows (element i: row r, column l + L i) and
  // as columns (row l + L i, column c).
  auto ex_row = [&](int p, unsigned r, unsigned l, int i) __attribute__((always_inline)) {
    return psi.far((size_t)p * NN * 8 + tile_idx<N>(0, L * i) * 8).at(tile_idx<N>(r, l) * 8);
  };
  auto ex_col = [&](int p, unsigned c, unsigned l, int i) __attribute__((always_inline)) {
    return psi.far((size_t)p * NN * 8 + tile_idx<N>(L * i, 0) * 8).at(tile_idx<N>(l, c) * 8);
  };
  // mode k of this wave
  auto mode = [&](int k) __attribute__((always_inline)) { return mw + MW * k; };
  auto has = [&](int k) __attribute__((always_inline)) { return k == 0 || k < nk; };
  auto fft_modes = [&](auto inv, float2 (*v)[PT], const Lane<N>& ln) __attribute__((always_inline)) {
    side_by_side<F, KM, 0, decltype(inv)::value>(f, v, ln.sc, (int)ln.l);
  };
  constexpr std::integral_constant<bool, false> fwd{};
  constexpr std::integral_constant<bool, true> bwd{};
  // the plane of floats q of a wave's LDS, four points g of a lane
  auto plane = [&](char* w, int q, int g) __attribute__((always_inline)) {
    return (v4*)(w + q * S::kSum + g * 1024) + lane;
  };

  float2 Pr[KM][PT];  // this wave's modes of the unit's probe rows
  float2 o[PT];       // the unit's box rows
  float Ps[PT];       // sum_p |P_p|^2, at the groups of points this wave updates the object at

  // The workgroup's columns of pattern jj into the LDS, straight from memory:
  // a wave's load takes 64 / COLS whole row segments of its workgroup's COLS
  // columns (a wave that loaded its own G columns would fetch each segment
  // several times), in flight without registers until the next barrier.  Row
  // k's columns are stored XORed by bits of k, which spreads a column over
  // the banks.
  const int lc = __builtin_ctz(min(UW * G, N));  // log2 COLS
  auto pat_slot = [&](unsigned k, unsigned c) __attribute__((always_inline)) {
    return (k << lc) + (c ^ (k & ((1u << lc) - 1)));
  };
  auto fetch_pattern = [&](int jj) __attribute__((always_inline)) {
    if (rank * UW >= NU) return;
    unsigned t = threadIdx.x & 63;
    asm volatile("" : "+v"(t));
    const Glob g = gI.far((size_t)jj * NN * 4 + (size_t)rank * (UW * G) * 4);
    for (int b = wave; b < (N << lc) >> 6; b += WV) {
      const unsigned e = b * 64 + t, k = e >> lc, c = (e ^ k) & ((1u << lc) - 1);
      __builtin_amdgcn_global_load_lds((const MRPIE_AS1 void*)g.at((k * N + c) * 4).p,
                                       (__attribute__((address_space(3))) void*)(s_pat + 64 * b), 4, 0, 0);
    }
  };
  fetch_pattern(0);

  // Sums over the modes of this wave's ps (and num) at four-point groups: all
  // waves of a unit write theirs, the one that updates group g reads them.
  // Calls done(g, num.x, num.y, ps) for the groups g of this wave.
  auto mode_sums = [&](auto with_num, const v4 (&nx)[GR], const v4 (&ny)[GR], const v4 (&ps)[GR],
                       auto done) __attribute__((always_inline)) {
    constexpr bool NUM = decltype(with_num)::value;
    if (MW > 1) {
      if (active) {
#pragma unroll
        for (int g = 0; g < GR; ++g) {
          if constexpr (NUM) {
            *plane(mine, 0, g) = nx[g];
            *plane(mine, 1, g) = ny[g];
          }
          *plane(mine, 2, g) = ps[g];
        }
      }
      lds_barrier();
    }
    if (!active) return;
    const auto group = [&](auto gc) __attribute__((always_inline)) {
      constexpr int g = decltype(gc)::value;
      if (g % MW != mw) return;
      v4 x{}, y{}, q;
      if (MW == 1) {
        if constexpr (NUM) {
          x = nx[g];
          y = ny[g];
        }
        q = ps[g];
      } else {
        char* w = lds + ul * MW * S::kWave;
        if constexpr (NUM) {
          x = *plane(w, 0, g);
          y = *plane(w, 1, g);
        }
        q = *plane(w, 2, g);
        for (int m = 1; m < MW; ++m) {
          w += S::kWave;
          if constexpr (NUM) {
            x += *plane(w, 0, g);
            y += *plane(w, 1, g);
          }
          q += *plane(w, 2, g);
        }
      }
      done(gc, x, y, q);
    };
    group(std::integral_constant<int, 0>{});
    group(std::integral_constant<int, 1>{});
    if constexpr (GR > 2) group(std::integral_constant<int, 2>{});
  };

  // the probe's rows, and the maximum of their sum over modes
  {
    v4 ps[GR];
    float m = 0.f;
    if (active) {
      const Lane<N> ln((float2*)mine);
#pragma unroll
      for (int g = 0; g < GR; ++g) ps[g] = v4{};
#pragma unroll
      for (int k = 0; k < KM; ++k)
        if (has(k)) {
          const Glob P = gprobe.far((size_t)mode(k) * NN * 8).at(((u * G + ln.grp) * N + ln.l) * 8);
#pragma unroll
          for (int i = 0; i < PT; ++i) Pr[k][i] = P.far(L * 8 * i).ld2();
        } else {
#pragma unroll
          for (int i = 0; i < PT; ++i) Pr[k][i] = mk(0.f, 0.f);
        }
#pragma unroll
      for (int k = 0; k < KM; ++k)
#pragma unroll
        for (int i = 0; i < PT; ++i) ps[i / 4][i % 4] = xadd_abs2(ps[i / 4][i % 4], Pr[k][i]);
    }
    mode_sums(std::false_type{}, ps, ps, ps, [&](auto gc, v4 sx, v4 sy, v4 sp) __attribute__((always_inline)) {
      constexpr int g = decltype(gc)::value;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        Ps[4 * g + e] = sp[e];
        m = fmaxf(m, sp[e]);
      }
    });
    sh->part[wave] = wave_max(m);
    barrier.epoch = 1;
  }
  float pmaxv = barrier(2);
  if (!barrier.ok()) return;

  const float invN = 1.0f / (float)N;
  float py = gpos.ld<float>(), px = gpos.far(4).ld<float>();  // the position ahead
  for (int it = 0; it < T; ++it) {
    const bool upd_p = cm.iter_offset + it >= cm.probe_update_start;
    double e = 0.0, isv = 0.0;  // this lane's share of the unit's error and intensity (waves of mode 0)
    for (int j = 0; j < J; ++j) {
      ++barrier.epoch;
      const int ny = __builtin_amdgcn_readfirstlane(box_corner(py, H - N, jb.status));
      const int nx = __builtin_amdgcn_readfirstlane(box_corner(px, W - N, jb.status));
      const int jn = j + 1 < J ? j + 1 : 0;  // the next position, loaded during the gather
      py = gpos.far((size_t)jn * 8).ld<float>();
      px = gpos.far((size_t)jn * 8 + 4).ld<float>();
      const Glob gbox = gobj.far(((size_t)ny * W + nx) * 8);
      bool bad = false;
      // ---- gather: rows of the box, exit waves, forward row FFTs
      float m = 0.f;
      if (active) {
        const Lane<N> ln((float2*)mine);
        const unsigned l = ln.l, r = u * G + ln.grp;
        const Glob ob = gbox.far(((size_t)r * W + l) * 8);
#pragma unroll
        for (int i = 0; i < PT; ++i) o[i] = ob.far(L * 8 * i).ld2_team();
        float2 v[KM][PT];
#pragma unroll
        for (int k = 0; k < KM; ++k)
#pragma unroll
          for (int i = 0; i < PT; ++i) v[k][i] = xmul(Pr[k][i], o[i]);
        fft_modes(fwd, v, ln);
#pragma unroll
        for (int k = 0; k < KM; ++k)
          if (has(k)) {
#pragma unroll
            for (int i = 0; i < PT; ++i) ex_row(mode(k), r, l, i).st2(v[k][i]);
          }
        if (mw == 0) {
#pragma unroll
          for (int i = 0; i < PT; ++i) m = fmaxf(m, xabs2(o[i]));
          m = wave_max(m);
        }
      }
      sh->part[wave] = m;
      const float omax = barrier(0);
      if (!barrier.ok()) return;
      // ---- columns: forward FFTs, modulus (Eq. 7; both transforms are
      //      unnormalised, so the scale carries one 1 / N), inverse FFTs
      unsigned touch_o = 0, touch_i = 0;
      {
        float2 v[KM][PT];
        float A[PT];  // sum over modes of |Psi_p|^2, then the scale of Eq. 7
        if (active) {
          const Lane<N> ln((float2*)mine);
          const unsigned l = ln.l, c = u * G + ln.grp;
#pragma unroll
          for (int k = 0; k < KM; ++k)
            if (has(k)) {
#pragma unroll
              for (int i = 0; i < PT; ++i) v[k][i] = ex_col(mode(k), c, l, i).ld2_team();
            } else {
#pragma unroll
              for (int i = 0; i < PT; ++i) v[k][i] = mk(0.f, 0.f);
            }
          // One word of each 128-byte line that the next position takes from
          // memory (the unit's box rows, an equal share of the pattern): the
          // lines come in while the columns are transformed, and the phases
          // that use them find them in the L2 (from memory the loads of a box
          // row took 1.9 us a position at 256^2 x 3, those of a pattern 1.3).
          constexpr unsigned RL = N * 8 / 128 + 1;  // lines of a row, which need not start on one
          constexpr unsigned PL = NN * 4 / 128;     // lines of a pattern
          static_assert(G * RL <= 64 && PL <= 64 * NU && PL % NU == 0, "one load each");
          unsigned t = threadIdx.x & 63;
          asm volatile("" : "+v"(t));
          if (mw == 0) {
            const int y = box_corner(py, H - N, nullptr), x = box_corner(px, W - N, nullptr);
            const unsigned tr = t < G * RL ? t : G * RL - 1, row = u * G + tr / RL, at = (tr % RL) * 128;
            touch_o = gobj.far(((size_t)y * W + x) * 8)
                          .far((size_t)row * W * 8 + (at < N * 8 ? at : N * 8 - 4))
                          .template ld<unsigned>();
          }
          if (mw == MW - 1) {
            constexpr unsigned per = PL / NU;
            touch_i = gI.far((size_t)jn * NN * 4).at((u * per + (t < per ? t : per - 1)) * 128).template ld<unsigned>();
          }
          fft_modes(fwd, v, ln);
#pragma unroll
          for (int i = 0; i < PT; ++i) A[i] = xabs2(v[0][i]);
#pragma unroll
          for (int k = 1; k < KM; ++k)
#pragma unroll
            for (int i = 0; i < PT; ++i) A[i] = xadd_abs2(A[i], v[k][i]);
          if (MW > 1) {
#pragma unroll
            for (int g = 0; g < GR; ++g)
              *plane(mine + S::kFft, 0, g) = v4{A[4 * g], A[4 * g + 1], A[4 * g + 2], A[4 * g + 3]};
          }
        }
        if (MW > 1) lds_barrier();
        if (active) {
          const Lane<N> ln((float2*)mine);
          const unsigned l = ln.l, c = u * G + ln.grp;
          if (MW > 1) {
            char* const w = lds + ul * MW * S::kWave + S::kFft;
#pragma unroll
            for (int g = 0; g < GR; ++g) {
              v4 s = *plane(w, 0, g);
              for (int q = 1; q < MW; ++q) s += *plane(w + q * S::kWave, 0, g);
#pragma unroll
              for (int x = 0; x < 4; ++x) A[4 * g + x] = s[x];
            }
          }
#pragma unroll
          for (int i = 0; i < PT; ++i) {
            const float Ic = fmaxf(s_pat[pat_slot(l + L * i, c - rank * (UW * G))], 0.f);
            const float rs = A[i] > 0.f ? __builtin_amdgcn_rsqf(A[i]) : 0.f;
            const float sq = __builtin_amdgcn_sqrtf(Ic);
            if (mw == 0) {
              const float d = xmisfit(A[i], rs, invN, sq);
              e += (double)d * (double)d;
              isv += (double)Ic;
              bad |= !isfinite(A[i]);
            }
            A[i] = sq * rs * invN;
          }
#pragma unroll
          for (int k = 0; k < KM; ++k)
#pragma unroll
            for (int i = 0; i < PT; ++i) v[k][i] = xscale(v[k][i], A[i]);
          fft_modes(bwd, v, ln);
#pragma unroll
          for (int k = 0; k < KM; ++k)
            if (has(k)) {
#pragma unroll
              for (int i = 0; i < PT; ++i) ex_col(mode(k), c, l, i).st2(v[k][i]);
            }
          if (mw == 0 && j == J - 1) {
            const size_t at = ((size_t)it * kErrSlots + u) * 8;
            gerr.far(at).template st<double>(wave_sum(e));
            gis.far(at).template st<double>(wave_sum(isv));
          }
        }
      }
      barrier(1);
      if (!barrier.ok()) return;
      asm volatile("" ::"v"(touch_o), "v"(touch_i));
      // ---- update: inverse row FFTs, probe rows, object rows.  The next
      //      pattern comes in meanwhile (a barrier waits for loads and stores
      //      alike, so it is there after the next one).
      fetch_pattern(jn);
      m = 0.f;
      {
        v4 nx[GR], ny[GR], ps[GR];
        if (active) {
          const Lane<N> ln((float2*)mine);
          const unsigned l = ln.l, r = u * G + ln.grp;
          float2 v[KM][PT];
#pragma unroll
          for (int k = 0; k < KM; ++k)
            if (has(k)) {
#pragma unroll
              for (int i = 0; i < PT; ++i) v[k][i] = ex_row(mode(k), r, l, i).ld2_team();
            } else {
#pragma unroll
              for (int i = 0; i < PT; ++i) v[k][i] = mk(0.f, 0.f);
            }
          float gP[PT];
#pragma unroll
          for (int i = 0; i < PT; ++i) {
            const float dP = xblend(cm.beta, omax, xabs2(o[i]));
            gP[i] = (upd_p && dP != 0.f) ? cm.alpha_probe / dP : 0.f;
          }
#pragma unroll
          for (int g = 0; g < GR; ++g) nx[g] = ny[g] = ps[g] = v4{};
          fft_modes(bwd, v, ln);
#pragma unroll
          for (int k = 0; k < KM; ++k)
#pragma unroll
            for (int i = 0; i < PT; ++i) {
              const float2 d = xnmac(v[k][i], Pr[k][i], o[i]);
              nx[i / 4][i % 4] = xadd_dot(nx[i / 4][i % 4], d, Pr[k][i]);
              ny[i / 4][i % 4] = xadd_cross(ny[i / 4][i % 4], d, Pr[k][i]);
              Pr[k][i] = xaxpy(Pr[k][i], xmulc(d, o[i]), gP[i]);
              ps[i / 4][i % 4] = xadd_abs2(ps[i / 4][i % 4], Pr[k][i]);
            }
        }
        mode_sums(std::true_type{}, nx, ny, ps, [&](auto gc, v4 sx, v4 sy, v4 sp) __attribute__((always_inline)) {
      constexpr int g = decltype(gc)::value;
          const Lane<N> ln((float2*)mine);
          const Glob ob = gbox.far(((size_t)(u * G + ln.grp) * W + ln.l) * 8);
#pragma unroll
          for (int x = 0; x < 4; ++x) {
            const int i = 4 * g + x;
            const float dO = xblend(cm.gamma, pmaxv, Ps[i]);
            const float gO = dO != 0.f ? cm.alpha_obj / dO : 0.f;
            const float2 on = xaxpy(o[i], mk(sx[x], sy[x]), gO);
            bad |= !(isfinite(on.x) && isfinite(on.y)) || !isfinite(sp[x]);
            ob.far(L * 8 * i).st2(on);
            Ps[i] = sp[x];
            m = fmaxf(m, sp[x]);
          }
        });
        sh->part[wave] = wave_max(m);
      }
      if (__builtin_amdgcn_ballot_w64(bad)) flag_status(jb.status, MRPIE_STATUS_NONFINITE);
      pmaxv = barrier(2);
      if (!barrier.ok()) return;
    }
    if (err_out && rank == 0 && wave == 0) iteration_error<NU>(gerr, gis, err_out, it);
  }
  if (active) {
    const Lane<N> ln((float2*)mine);
#pragma unroll
    for (int k = 0; k < KM; ++k)
      if (has(k)) {
        const Glob P = gprobe.far((size_t)mode(k) * NN * 8).at(((u * G + ln.grp) * N + ln.l) * 8);
#pragma unroll
        for (int i = 0; i < PT; ++i) P.far(L * 8 * i).st2(Pr[k][i]);
      }
  }
}

// ... by a team with fewer waves: every wave takes its units of a phase in
// turn, mode by mode, with the probe, the sums and the error in memory.  Only
// a launch that found the GPU busy gets here (or one told to form small teams:
// mrpie_team_sweep); sums are taken in run_units' order.
template <int N, int KM, int WV>
__device__ __forceinline__ void run_loops(const Common& cm, const JobRec& jb, float* err_out, int rank, int size,
                                          char* lds, Shared* sh) {
  using F = WaveFft<N>;
  constexpr int L = F::L, PT = F::PT, G = F::G, NU = N / G;
  constexpr unsigned NN = N * N;
  const int M = jb.M, MW = (M + KM - 1) / KM, J = jb.J, T = jb.T, H = jb.H, W = jb.W;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int w0 = rank * WV + wave, nw = size * WV;
  const WsLayout ly = ws_layout(N, M, T);
  const Glob gobj(jb.obj), gprobe(jb.probe), gpos(jb.pos), gI(jb.I), ws(jb.ws);
  const Glob psi = ws.far(ly.psi[0]), gerr = ws.far(ly.err), gis = ws.far(ly.isum);
  const Glob shares = ws.far(ly.patch[0]);  // a lane's share of a unit's error and intensity
  JobBarrier<WV> barrier{ws.far(ly.psi[1] + kFlagOffset), rank, size, sh, __builtin_amdgcn_readfirstlane(sh->spin)};
  char* const lds0 = lds;
  float2* const wsc = (float2*)(lds + TeamLds<N, WV>::kHead) + wave * F::SCRATCH;
  F f;
  init_fft<N>(f, (float2*)(lds0 + TeamLds<N, WV>::kPat));
  auto ex = [&](int p, unsigned k, unsigned c) __attribute__((always_inline)) {
    return psi.far((size_t)p * NN * 8).at(tile_idx<N>(k, c) * 8);
  };
  auto probe = [&](int p, unsigned r, unsigned l, int i) __attribute__((always_inline)) {
    return gprobe.far((size_t)p * NN * 8 + L * 8 * i).at((r * N + l) * 8);
  };
  float m = 0.f;
  for (int u = w0; u < NU; u += nw) {
    const Lane<N> ln(wsc);
    float s[PT];
#pragma unroll
    for (int i = 0; i < PT; ++i) s[i] = 0.f;
    for (int q = 0; q < MW; ++q) {
      float t[PT];
#pragma unroll
      for (int i = 0; i < PT; ++i) t[i] = 0.f;
      for (int p = q; p < M; p += MW)
#pragma unroll
        for (int i = 0; i < PT; ++i) t[i] = xadd_abs2(t[i], probe(p, u * G + ln.grp, ln.l, i).ld2());
#pragma unroll
      for (int i = 0; i < PT; ++i) s[i] += t[i];
    }
#pragma unroll
    for (int i = 0; i < PT; ++i) m = fmaxf(m, s[i]);
  }
  sh->part[wave] = wave_max(m);
  barrier.epoch = 1;
  float pmaxv = barrier(2);
  if (!barrier.ok()) return;
  const float invN = 1.0f / (float)N;
  for (int it = 0; it < T; ++it) {
    const bool upd_p = cm.iter_offset + it >= cm.probe_update_start;
    for (int j = 0; j < J; ++j) {
      ++barrier.epoch;
      const int ny = __builtin_amdgcn_readfirstlane(box_corner(gpos.far((size_t)j * 8).ld<float>(), H - N, jb.status));
      const int nx =
          __builtin_amdgcn_readfirstlane(box_corner(gpos.far((size_t)j * 8 + 4).ld<float>(), W - N, jb.status));
      const Glob gbox = gobj.far(((size_t)ny * W + nx) * 8);
      bool bad = false;
      float m = 0.f;
      for (int u = w0; u < NU; u += nw) {
        const Lane<N> ln(wsc);
        const unsigned l = ln.l, r = u * G + ln.grp;
        const Glob ob = gbox.far(((size_t)r * W + l) * 8);
        float2 o[PT];
#pragma unroll
        for (int i = 0; i < PT; ++i) {
          o[i] = ob.far(L * 8 * i).ld2_team();
          m = fmaxf(m, xabs2(o[i]));
        }
        for (int p = 0; p < M; ++p) {
          float2 v[1][PT];
#pragma unroll
          for (int i = 0; i < PT; ++i) v[0][i] = xmul(probe(p, r, l, i).ld2(), o[i]);
          f.template run<1, false>(v, ln.sc, (int)l);
#pragma unroll
          for (int i = 0; i < PT; ++i) ex(p, r, l + L * i).st2(v[0][i]);
        }
      }
      sh->part[wave] = wave_max(m);
      const float omax = barrier(0);
      if (!barrier.ok()) return;
      for (int u = w0; u < NU; u += nw) {
        const Lane<N> ln(wsc);
        const unsigned l = ln.l, c = u * G + ln.grp;
        float A[PT];
#pragma unroll
        for (int i = 0; i < PT; ++i) A[i] = 0.f;
        for (int q = 0; q < MW; ++q) {
          float t[PT];
#pragma unroll
          for (int i = 0; i < PT; ++i) t[i] = 0.f;
          for (int p = q; p < M; p += MW) {
            float2 v[1][PT];
#pragma unroll
            for (int i = 0; i < PT; ++i) v[0][i] = ex(p, l + L * i, c).ld2_team();
            f.template run<1, false>(v, ln.sc, (int)l);
#pragma unroll
            for (int i = 0; i < PT; ++i) {
              t[i] = xadd_abs2(t[i], v[0][i]);
              ex(p, l + L * i, c).st2(v[0][i]);
            }
          }
#pragma unroll
          for (int i = 0; i < PT; ++i) A[i] += t[i];
        }
        const Glob g = gI.far((size_t)j * NN * 4).at((l * N + c) * 4);
        const Glob es = shares.at((u * 64 + lane) * 16);
        double e = j ? es.ld<double>() : 0.0, isv = j ? es.far(8).ld<double>() : 0.0;
#pragma unroll
        for (int i = 0; i < PT; ++i) {
          const float Ic = fmaxf(g.far(L * N * 4 * i).template ld<float>(), 0.f);
          const float rs = A[i] > 0.f ? __builtin_amdgcn_rsqf(A[i]) : 0.f;
          const float sq = __builtin_amdgcn_sqrtf(Ic);
          const float d = xmisfit(A[i], rs, invN, sq);
          e += (double)d * (double)d;
          isv += (double)Ic;
          bad |= !isfinite(A[i]);
          A[i] = sq * rs * invN;
        }
        es.st<double>(e);
        es.far(8).st<double>(isv);
        if (j == J - 1) {
          const size_t at = ((size_t)it * kErrSlots + u) * 8;
          gerr.far(at).template st<double>(wave_sum(e));
          gis.far(at).template st<double>(wave_sum(isv));
        }
        // the lane reads back what it stored: no other member writes it
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        for (int p = 0; p < M; ++p) {
          float2 v[1][PT];
#pragma unroll
          for (int i = 0; i < PT; ++i) v[0][i] = xscale(ex(p, l + L * i, c).ld2_team(), A[i]);
          f.template run<1, true>(v, ln.sc, (int)l);
#pragma unroll
          for (int i = 0; i < PT; ++i) ex(p, l + L * i, c).st2(v[0][i]);
        }
      }
      barrier(1);
      if (!barrier.ok()) return;
      m = 0.f;
      for (int u = w0; u < NU; u += nw) {
        const Lane<N> ln(wsc);
        const unsigned l = ln.l, r = u * G + ln.grp;
        const Glob ob = gbox.far(((size_t)r * W + l) * 8);
        float2 o[PT], num[PT];
        float gP[PT], Ps[PT], ps[PT];
#pragma unroll
        for (int i = 0; i < PT; ++i) {
          o[i] = ob.far(L * 8 * i).ld2_team();
          const float dP = xblend(cm.beta, omax, xabs2(o[i]));
          gP[i] = (upd_p && dP != 0.f) ? cm.alpha_probe / dP : 0.f;
          num[i] = mk(0.f, 0.f);
          Ps[i] = ps[i] = 0.f;
        }
        for (int q = 0; q < MW; ++q) {
          float2 tn[PT];
          float tP[PT], tp[PT];
#pragma unroll
          for (int i = 0; i < PT; ++i) {
            tn[i] = mk(0.f, 0.f);
            tP[i] = tp[i] = 0.f;
          }
          for (int p = q; p < M; p += MW) {
            float2 v[1][PT];
#pragma unroll
            for (int i = 0; i < PT; ++i) v[0][i] = ex(p, r, l + L * i).ld2_team();
            f.template run<1, true>(v, ln.sc, (int)l);
#pragma unroll
            for (int i = 0; i < PT; ++i) {
              float2 P = probe(p, r, l, i).ld2();
              tP[i] = xadd_abs2(tP[i], P);
              const float2 d = xnmac(v[0][i], P, o[i]);
              tn[i] = mk(xadd_dot(tn[i].x, d, P), xadd_cross(tn[i].y, d, P));
              P = xaxpy(P, xmulc(d, o[i]), gP[i]);
              tp[i] = xadd_abs2(tp[i], P);
              probe(p, r, l, i).st2(P);
            }
          }
#pragma unroll
          for (int i = 0; i < PT; ++i) {
            num[i] = cadd(num[i], tn[i]);
            Ps[i] += tP[i];
            ps[i] += tp[i];
          }
        }
#pragma unroll
        for (int i = 0; i < PT; ++i) {
          const float dO = xblend(cm.gamma, pmaxv, Ps[i]);
          const float gO = dO != 0.f ? cm.alpha_obj / dO : 0.f;
          const float2 on = xaxpy(o[i], num[i], gO);
          bad |= !(isfinite(on.x) && isfinite(on.y)) || !isfinite(ps[i]);
          ob.far(L * 8 * i).st2(on);
          m = fmaxf(m, ps[i]);
        }
      }
      sh->part[wave] = wave_max(m);
      if (__builtin_amdgcn_ballot_w64(bad)) flag_status(jb.status, MRPIE_STATUS_NONFINITE);
      pmaxv = barrier(2);
      if (!barrier.ok()) return;
    }
    if (err_out && w0 == 0) iteration_error<NU>(gerr, gis, err_out, it);
  }
}

// ------------------------------------------------------------------ teams
// The next job of class c, -1 when all are taken.
__device__ __forceinline__ int pop_job(const TeamArgs& a, int c) {
  const int n = a.first[c + 1] - a.first[c];
  if (ld_agent(a.ctrl + c) >= (unsigned)n) return -1;
  const unsigned k = add_agent(a.ctrl + c, 1u);
  return k < (unsigned)n ? a.first[c] + (int)k : -1;
}

// A job as scalars: the record is not written during the launch, and read
// through a generic pointer its fields would count as different in each lane.
__device__ __forceinline__ JobRec job_of(const TeamJob* t) {
  const MRPIE_AS4 JobRec* j = &((const MRPIE_AS4 TeamJob*)(unsigned long long)t)->j;
  JobRec r;
  r.obj = j->obj;
  r.probe = j->probe;
  r.pos = j->pos;
  r.I = j->I;
  r.ws = j->ws;
  r.status = j->status;
  r.H = j->H;
  r.W = j->W;
  r.N = j->N;
  r.M = j->M;
  r.J = j->J;
  r.T = j->T;
  return r;
}

// Largest number of modes a wave takes (the register budget of 8 waves).
constexpr int max_km(int N) { return N == 256 ? 3 : N == 32 ? 1 : 2; }

using LdsChar = __attribute__((address_space(3))) char*;
using LdsShared = __attribute__((address_space(3))) Shared*;

// One job for one member, as a function of its own: each probe size and
// schedule gets its own register allocation.  Arguments arrive in vector
// registers.
template <int N, int KM, bool LOOPS, int WV>
__device__ __attribute__((noinline)) void member_job(unsigned long long t, int rank, int size, LdsChar lds,
                                                     LdsShared sh) {
  const auto uni = [](unsigned long long v) {
    return (unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)v) |
           (unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32;
  };
  const MRPIE_AS4 TeamJob* tj = (const MRPIE_AS4 TeamJob*)uni(t);
  const JobRec jb = job_of((const TeamJob*)uni(t));
  Common c;
  c.alpha_obj = tj->c.alpha_obj;
  c.alpha_probe = tj->c.alpha_probe;
  c.beta = tj->c.beta;
  c.gamma = tj->c.gamma;
  c.iter_offset = tj->c.iter_offset;
  c.probe_update_start = tj->c.probe_update_start;
  rank = __builtin_amdgcn_readfirstlane(rank);
  size = __builtin_amdgcn_readfirstlane(size);
  if constexpr (LOOPS) run_loops<N, KM, WV>(c, jb, tj->err_out, rank, size, (char*)lds, (Shared*)sh);
  else run_units<N, KM, WV>(c, jb, tj->err_out, rank, size, (char*)lds, (Shared*)sh);
}

template <int N, int KM, int WV>
__device__ __forceinline__ void member(const TeamJob* t, int M, const Team& tm, char* lds, Shared* sh) {
  const Deal<N, KM, WV> d(M, tm.size);
  if (d.fits(tm.size)) {
    const int n = d.members();
    if (tm.rank < n)
      member_job<N, KM, false, WV>((unsigned long long)t, tm.rank, n, (LdsChar)lds, (LdsShared)sh);
  } else {
    member_job<N, KM, true, WV>((unsigned long long)t, tm.rank, tm.size, (LdsChar)lds, (LdsShared)sh);
  }
}

// A team that leaves: of the jobs that it might have run after this one, its
// leader flags those that no other team has taken.
__device__ __forceinline__ void give_up(const TeamArgs& a, const Team& tm, int c) {
  if (tm.rank != 0 || threadIdx.x != 0) return;
  for (; c < kClasses; ++c)
    for (int q; (q = pop_job(a, c)) >= 0;) flag_status(a.job[q]->j.status, MRPIE_STATUS_UNFINISHED);
}

// N: the probe size of every job of the launch, 0: any mix.
template <int N, int WV>
__global__ __launch_bounds__(WV * 64, WV / 4) void k_team(const TeamArgs a) {
  extern __shared__ __align__(16) char lds[];
  __shared__ Shared sh;
  // workgroups go to the XCDs in turn
  if ((blockIdx.x + (unsigned)(a.nxcc - a.from)) % (unsigned)a.nxcc >= (unsigned)a.xccs) return;
  const int x = xcc_id();
  unsigned* const ctrl = a.ctrl + kCtrlXcc + x * kXccWords;
  if (threadIdx.x == 0) {
    sh.ok = 1;
    sh.spin = a.spin;
    // arrive; the first on this XCD closes the list
    const unsigned t = add_agent(ctrl, 1u);
    unsigned n = 0;
    const long long t0 = wall_clock64();
    if (t == 0) {
      while (ld_agent(ctrl) < (unsigned)a.expect && wall_clock64() - t0 < kFormTicks) {
      }
      n = __hip_atomic_fetch_or(ctrl, kClosed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      st_agent(ctrl + 1, n | kClosed);
    } else if (!(t & kClosed)) {
      while (!((n = ld_agent(ctrl + 1)) & kClosed) && wall_clock64() - t0 < kIdleTicks) {
      }
      n &= ~kClosed;
    }
    sh.rank = (int)t;
    sh.size = (t & kClosed) ? 0 : min((int)n, a.limit);
  }
  __syncthreads();
  const int me = __builtin_amdgcn_readfirstlane(sh.rank), there = __builtin_amdgcn_readfirstlane(sh.size);
  if (me >= there) return;  // late (or the list never closed)
  for (int c = 0; c < kClasses; ++c) {
    if (a.first[c + 1] == a.first[c]) continue;
    const int cap = kMaxSize >> c, team = me / cap;
    Team tm{me - team * cap, min(cap, there - team * cap), ctrl + 2 + 4 * ((1 << c) - 1 + team), 0u};
    if (team >= 1 << c) continue;  // more workgroups than teams
    for (;;) {
      if (tm.rank == 0 && threadIdx.x == 0) st_agent(tm.bar + 2, (unsigned)pop_job(a, c));
      if (!team_barrier(tm, &sh)) return give_up(a, tm, c);
      const int q = (int)ld_uniform(tm.bar + 2);
      if (q < 0) break;
      const TeamJob* t = a.job[q];
      const MRPIE_AS4 TeamJob* tj = (const MRPIE_AS4 TeamJob*)(unsigned long long)t;
      const int M = tj->j.M, km = tj->km;
      const auto go = [&](auto n) __attribute__((always_inline)) {
        constexpr int NN = decltype(n)::value, most = WV == 8 ? max_km(NN) : 1;
        if (km == 1) member<NN, 1, WV>(t, M, tm, lds, &sh);
        if constexpr (most >= 2) {
          if (km == 2) member<NN, 2, WV>(t, M, tm, lds, &sh);
        }
        if constexpr (most >= 3) {
          if (km == 3) member<NN, 3, WV>(t, M, tm, lds, &sh);
        }
      };
      switch (N ? N : tj->j.N) {
        case 32: go(std::integral_constant<int, N ? N : 32>{}); break;
        case 64: go(std::integral_constant<int, N ? N : 64>{}); break;
        case 128: go(std::integral_constant<int, N ? N : 128>{}); break;
        case 192: go(std::integral_constant<int, N ? N : 192>{}); break;
        default: go(std::integral_constant<int, N ? N : 256>{}); break;
      }
      // (every member is past the job's last barrier before the leader's next
      // pop is read, and reads tm.bar + 2 before it can arrive at that barrier)
      if (!__builtin_amdgcn_readfirstlane(sh.ok)) {
        st_agent(tm.bar + 1, tm.target + (unsigned)tm.size);
        flag_status(tj->j.status, MRPIE_STATUS_UNFINISHED);
      }
      if (!team_barrier(tm, &sh)) return give_up(a, tm, c);
    }
  }
}

struct SetupArgs {
  LaunchArgs a;
  float* err_out[kMaxJobsPerLaunch];
  unsigned char km[kMaxJobsPerLaunch];
  unsigned* ctrl;  // cleared when set
};
static_assert(sizeof(SetupArgs) <= 4096, "kernel arguments");

// One workgroup per job: its record and flags; the first clears the control
// words too.
__global__ __launch_bounds__(256) void k_team_setup(const SetupArgs s) {
  if (s.ctrl && blockIdx.x == 0)
    for (int i = threadIdx.x; i < (int)(kCtrlBytes / 4); i += 256) s.ctrl[i] = 0;
  const JobRec& jb = s.a.job[blockIdx.x];
  char* p = jb.ws + ws_layout(jb.N, jb.M, jb.T).psi[1];
  for (int i = threadIdx.x; i < kFlagWords; i += 256) ((unsigned*)(p + kFlagOffset))[i] = 0;
  if (threadIdx.x == 0) {
    TeamJob* t = (TeamJob*)(p + kJobOffset);
    t->j = jb;
    t->err_out = s.err_out[blockIdx.x];
    t->c = s.a.c;
    t->km = s.km[blockIdx.x];
  }
}

using TeamKernel = void (*)(const TeamArgs);
struct TeamLaunch {
  TeamKernel k;
  size_t lds;
};
// The kernel of jobs of N^2 probes (0: any mix) and its waves.  Three modes
// of 256^2 take 12 waves a workgroup, one for each mode of four units.
TeamLaunch team_kernel(int N, int waves) {
  if (waves == 12) return {k_team<256, 12>, TeamLds<256, 12>::kBytes};
  switch (N) {
    case 32: return {k_team<32, 8>, TeamLds<32, 8>::kBytes};
    case 64: return {k_team<64, 8>, TeamLds<64, 8>::kBytes};
    case 128: return {k_team<128, 8>, TeamLds<128, 8>::kBytes};
    case 192: return {k_team<192, 8>, TeamLds<192, 8>::kBytes};
    case 256: return {k_team<256, 8>, TeamLds<256, 8>::kBytes};
    default:
      return {k_team<0, 8>, (size_t)std::max({TeamLds<32, 8>::kBytes, TeamLds<64, 8>::kBytes, TeamLds<128, 8>::kBytes,
                                              TeamLds<192, 8>::kBytes, TeamLds<256, 8>::kBytes})};
  }
}

// Members that hold a job whose waves take km modes: units / units of a full
// workgroup.
int job_need(int N, int M, int waves, int km) {
  const int G = N == 256 ? 2 : N == 192 || N == 128 ? 4 : N == 64 ? 8 : 16;
  const int mw = (M + km - 1) / km;
  if (mw > waves) return kMaxSize + 1;
  int uw = 1;
  while (uw * 2 * mw <= waves) uw *= 2;
  return (N / G + uw - 1) / uw;
}
// Members that take part in it: as many as its units keep busy (Deal's); but
// 32^2 x 1 is one workgroup's (5.65 us a position, by two 5.95; x 2 6.57 / 6.35,
// 64^2 x 1 by one 9.67, by eight 6.40).
int job_members(int N, int M, int waves, int km) {
  if (N == 32 && M == 1) return 1;
  const int G = N == 256 ? 2 : N == 192 || N == 128 ? 4 : N == 64 ? 8 : 16, mw = (M + km - 1) / km;
  int uw = 1;
  while (uw * 2 * mw <= waves && uw * kMaxSize < N / G) uw *= 2;
  return (N / G + uw - 1) / uw;
}
// Modes of a wave: as few as let a team of `cap` hold the job, or as few as
// any team can.
int job_km(int N, int M, int waves, int cap) {
  const int most = waves == 8 ? max_km(N) : 1;
  for (; cap <= kMaxSize; cap *= 2)
    for (int km = 1; km <= most; ++km)
      if (job_need(N, M, waves, km) <= cap) return km;
  return 0;
}

}  // namespace


// Launches on the same XCD run one at a time: two that each held half of its
// CUs would wait for members until their lists close.  A call of fewer jobs
// than XCDs takes one XCD for each, so calls on several streams run side by
// side: a stream keeps the XCDs it last used, or takes idle ones, or queues
// behind the last launch on others, the highest first: workgroups go to the
// XCDs in turn from the first, so kernels of a few workgroups (the next call's
// setup among them) find room on the lower ones.  An event of each launch is kept for the
// XCDs that it was the last on.
namespace {
constexpr int kMaxDevices = 16;  // (on further ones nothing is queued)
struct Turns {
  hipEvent_t ev[kMaxXcc + 1] = {};
  int last[kMaxXcc];             // event of the last launch on each XCD, -1: none
  hipStream_t by[kMaxXcc] = {};  // its stream, only ever compared
  unsigned next = 0;             // taken downwards from here
  bool ready = false;
};
Turns g_turns[kMaxDevices];
std::mutex g_turns_mu;

int init_turns(Turns& t) {
  if (t.ready) return MRPIE_OK;
  for (hipEvent_t& e : t.ev)
    if (!e) MRPIE_HIP(hipEventCreateWithFlags(&e, hipEventDisableTiming));
  std::fill(t.last, t.last + kMaxXcc, -1);
  t.ready = true;
  return MRPIE_OK;
}

// The first of `n` adjacent XCDs for a launch on `s`.
int pick_xccs(Turns& t, int n, int nxcc, hipStream_t s) {
  const auto own = [&](int x) { return t.last[x] >= 0 && t.by[x] == s; };
  int cost[kMaxXcc];
  for (int i = 0; i < nxcc; ++i) {
    bool all = true;
    for (int k = 0; k < n; ++k) all &= own((i + k) % nxcc);
    if (all) return i;
  }
  // (an event may be queried while another thread captures a graph)
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  (void)hipThreadExchangeStreamCaptureMode(&mode);
  for (int x = 0; x < nxcc; ++x)
    cost[x] = own(x) ? 0 : t.last[x] < 0 || hipEventQuery(t.ev[t.last[x]]) == hipSuccess ? 1 : 2 * nxcc;
  (void)hipThreadExchangeStreamCaptureMode(&mode);
  if (hipPeekAtLastError() == hipErrorNotReady) (void)hipGetLastError();  // it is none
  int best = 0, least = INT32_MAX;
  for (int i = 0; i < nxcc; ++i) {
    const int from = (int)((t.next + 2 * nxcc - n - i) % nxcc);
    int c = 0;
    for (int k = 0; k < n; ++k) c += cost[(from + k) % nxcc];
    if (c < least) {
      least = c;
      best = from;
    }
  }
  t.next = (unsigned)best;
  return best;
}

// Queues `s` behind the last launches on those XCDs.
int wait_turn(const Turns& t, int from, int n, int nxcc, hipStream_t s) {
  unsigned waited = 0;
  for (int k = 0; k < n; ++k) {
    const int e = t.last[(from + k) % nxcc];
    if (e < 0 || (waited >> e & 1)) continue;
    waited |= 1u << e;
    MRPIE_HIP(hipStreamWaitEvent(s, t.ev[e], 0));
  }
  return MRPIE_OK;
}

// What was launched on `s` is the last on them.
int record_turn(Turns& t, int from, int n, int nxcc, hipStream_t s) {
  unsigned used = 0;
  for (int k = 0; k < n; ++k) t.last[(from + k) % nxcc] = -1;
  for (int x = 0; x < nxcc; ++x)
    if (t.last[x] >= 0) used |= 1u << t.last[x];
  const int e = __builtin_ctz(~used);
  MRPIE_HIP(hipEventRecord(t.ev[e], s));
  for (int k = 0; k < n; ++k) {
    t.last[(from + k) % nxcc] = e;
    t.by[(from + k) % nxcc] = s;
  }
  return MRPIE_OK;
}
}  // namespace

// Whether a call of `njobs` jobs, of this size each, is for the teams rather
// than the launches of sweep.hip.  Measured in us a position of the card
// (launches / team), whole calls of 8 to 64 positions a job, every M from 1 to
// 8 and 1 to 64 jobs:
//   32^2, 64^2, 128^2  teams faster throughout: singles 64^2 x 1 10.2 / 6.8,
//       128^2 x 3 12.2 / 9.0, x 8 17.5 / 12.6; least at 20 to 64 jobs of 128^2
//       with many modes: 40 x 5 1.71 / 1.53, 64 x 5 1.70 / 1.61
//   256^2  x 3: single 16.3 / 14.6, 8 jobs 4.23 / 1.92, 9 3.79 / 3.29 (two to a
//       team on one XCD), 40 3.22 / 2.72; x 4: single 18.3 / 17.5; x 5 and x 6
//       (waves take three modes and spill): single 21.6 / 25.0 and 23.2 / 27.3,
//       2 jobs 14.2 / 12.6, 3 10.1 / 8.4, 9 6.37 / 5.86, 20 4.72 / 4.68
//   192^2  (48 units of 12 points a lane leave CUs idle)  single x 3 14.4 /
//       16.2; x 3 2 jobs 9.8 / 8.2, 8 3.13 / 2.11, 9 2.89 / 3.85, 16 2.25 / 2.27,
//       32 1.92 / 2.42; x 4 8 3.58 / 2.34, 9 3.33 / 3.97; x 5 2 12.5 / 13.9, 5
//       5.52 / 5.70, 8 4.18 / 3.56, 9 3.80 / 6.09.  (Up to 16 jobs x 2 and up to
//       32 x 1 the teams would win as well: 16 x 2 1.94 / 1.25, 32 x 1 1.13 /
//       0.71; two 256^2 x 5 and 8 jobs of 192^2 x 5 likewise.)
// For calls of mixed sizes see choose_team.
bool team_suits(int N, int M, int njobs) {
  if (N == 192) return M <= 4 && njobs >= 2 && njobs <= 8;
  if (N == 256) return M <= 4 || (M <= 6 && njobs > 2);
  return true;
}

bool team_fits(int N, int M) { return job_km(N, M, N == 256 && M == 3 ? 12 : 8, kMaxSize) > 0; }

int run_team(const Common& c, const JobRec* jobs, int njobs, float* const* err_out, hipStream_t s, int limit,
             int wait_ns) {
  if (njobs > kMaxTeamJobs) {
    for (int b = 0; b < njobs; b += kMaxTeamJobs) {
      const int rc = run_team(c, jobs + b, std::min(kMaxTeamJobs, njobs - b), err_out ? err_out + b : nullptr, s, limit,
                              wait_ns);
      if (rc) return rc;
    }
    return MRPIE_OK;
  }
  int dev = 0, cus = 0;
  MRPIE_HIP(hipGetDevice(&dev));
  MRPIE_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
  const int nxcc = std::min(kMaxXcc, std::max(1, cus / 32));
  // A launch holds its members' CUs, so it ends after about 15 ms' work (or an
  // iteration, if that is longer) and lets other streams' kernels in; the next
  // resumes with the same bits.
  long long longest = 1, all = 0;
  int T = 0;
  for (int b = 0; b < njobs; ++b) {
    longest = std::max<long long>(longest, jobs[b].J);
    all += jobs[b].J;
    T = std::max(T, jobs[b].T);
  }
  const int most = (int)std::max<long long>(1, kMaxPositions / std::max(longest, all / nxcc));
  if (T > most) {
    std::vector<JobRec> part(njobs);
    std::vector<float*> err(njobs);
    for (int it = 0; it < T; it += most) {
      Common ci = c;
      ci.iter_offset += it;
      int n = 0;
      for (int b = 0; b < njobs; ++b) {
        if (jobs[b].T <= it) continue;
        part[n] = jobs[b];
        part[n].T = std::min(most, jobs[b].T - it);
        err[n++] = err_out && err_out[b] ? err_out[b] + it : nullptr;
      }
      const int rc = run_team(ci, part.data(), n, err.data(), s, limit, wait_ns);
      if (rc) return rc;
    }
    return MRPIE_OK;
  }
  // A job's class: a team of 32, or as much smaller as it takes to give every
  // job of the call a team and as still holds it.
  int spare = 0;
  while (spare + 1 < kClasses && nxcc << spare < njobs) ++spare;
  std::vector<int> order(njobs), cls(njobs), km(njobs);
  int N = jobs[0].N, waves = 12;
  auto job_cost = [&](int b) {
    return (double)jobs[b].J * jobs[b].T * ((double)jobs[b].M * jobs[b].N * jobs[b].N + 40000.0);
  };
  for (int b = 0; b < njobs; ++b) {
    order[b] = b;
    if (jobs[b].N != N) N = 0;
    if (jobs[b].N != 256 || jobs[b].M != 3) waves = 8;
  }
  for (int b = 0; b < njobs; ++b) {
    km[b] = job_km(jobs[b].N, jobs[b].M, waves, kMaxSize >> spare);
    const int need = job_need(jobs[b].N, jobs[b].M, waves, km[b]);
    int k = spare;
    while (k > 0 && (kMaxSize >> k) < need) --k;
    cls[b] = k;
  }
  std::stable_sort(order.begin(), order.end(),
                   [&](int p, int q) { return cls[p] != cls[q] ? cls[p] < cls[q] : job_cost(p) > job_cost(q); });
  TeamArgs a{};
  for (int i = 0; i < njobs; ++i) {
    const JobRec& jb = jobs[order[i]];
    char* p = jb.ws + ws_layout(jb.N, jb.M, jb.T).psi[1];
    if (i == 0) a.ctrl = (unsigned*)p;
    a.job[i] = (const TeamJob*)(p + kJobOffset);
    a.first[cls[order[i]] + 1] = i + 1;
  }
  for (int k = 1; k <= kClasses; ++k) a.first[k] = std::max(a.first[k], a.first[k - 1]);
  // A call with an XCD for every job needs no more workgroups than its jobs'
  // members, and leaves the other CUs and XCDs free.
  a.nxcc = nxcc;
  a.xccs = std::min(njobs, nxcc);
  a.expect = kMaxSize;
  if (njobs <= nxcc) {
    a.expect = 1;
    for (int b = 0; b < njobs; ++b)
      a.expect = std::max(a.expect, job_members(jobs[b].N, jobs[b].M, waves, km[b]));
  }
  a.limit = limit;
  a.spin = wait_ns ? (int)((wait_ns + 9LL) / 10) : kSpinTicks;  // ticks of 10 ns
  const TeamLaunch tl = team_kernel(N, waves);
  MRPIE_HIP(ensure_lds((const void*)tl.k, tl.lds));
  int rc = launch_init_twiddles(s, n_index(N));
  if (rc) return rc;
  // (A stream under capture can't wait for work outside its graph; captured
  // launches take the XCDs in turn.)
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  MRPIE_HIP(hipStreamIsCapturing(s, &cap));
  const bool queue = cap == hipStreamCaptureStatusNone && dev < kMaxDevices;
  Turns& turns = g_turns[dev < kMaxDevices ? dev : 0];
  std::unique_lock<std::mutex> lk(g_turns_mu);
  if (queue) {
    rc = init_turns(turns);
    if (rc) return rc;
    a.from = pick_xccs(turns, a.xccs, nxcc, s);
    rc = wait_turn(turns, a.from, a.xccs, nxcc, s);
    if (rc) return rc;
  } else {
    a.from = (int)((turns.next + 2 * nxcc - a.xccs) % nxcc);
    turns.next = (unsigned)a.from;
    lk.unlock();
  }
  for (int b = 0; b < njobs; b += kMaxJobsPerLaunch) {
    SetupArgs u{};
    u.a.c = c;
    u.a.njobs = std::min(kMaxJobsPerLaunch, njobs - b);
    for (int k = 0; k < u.a.njobs; ++k) {
      u.a.job[k] = jobs[b + k];
      u.err_out[k] = err_out ? err_out[b + k] : nullptr;
      u.km[k] = (unsigned char)km[b + k];
    }
    u.ctrl = b == 0 ? a.ctrl : nullptr;
    hipLaunchKernelGGL(k_team_setup, dim3(u.a.njobs), dim3(256), 0, s, u);
  }
  long long positions = 0;
  for (int b = 0; b < njobs; ++b) positions += (long long)jobs[b].J * jobs[b].T;
  launch_ku(TK_TEAM, (int)std::min<long long>(positions, INT32_MAX), tl.k, dim3(a.expect * nxcc), dim3(waves * 64), tl.lds, s, a);
  MRPIE_HIP(hipGetLastError());
  return queue ? record_turn(turns, a.from, a.xccs, nxcc, s) : MRPIE_OK;
}

}  // namespace mrpie
