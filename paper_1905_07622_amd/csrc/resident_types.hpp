// Records and limits of the resident form (resident.hpp) that its host side
// shares with the kernels.
#pragma once

#include "common.hpp"
#include "solver.hpp"

namespace femheat {

constexpr int kResThreads = 512;   // most threads of a block (two waves per SIMD: 256 registers each)
constexpr int kResBlocks = 256;    // most blocks of a simulation (one per CU)
constexpr int kResHalo = 5;        // most halo nodes per thread
constexpr int kResRep = 8;         // copies of each partial
constexpr size_t kResLds = 160 * 1024 - 1024;  // dynamic LDS of a block (the rest: sums and flags)

// Polls before a wait gives up (about 0.7 us each).  The meeting: 20 ms in
// which no simulation of the launch runs.  Any other wait: 2 s.
constexpr uint32_t kResMeet = 30000, kResSpin = 3000000;

// What a launch does before it gives its compute units back: that many steps
// of a simulation, or fewer once it has lasted that long: its simulations then
// end at the end of the step they are in, and those whose turn has not come
// begin the next launch.  Other work on the device waits for a launch as a
// whole (a run of 1M nodes leaves it four compute units), and a server takes
// cancellations and admissions between launches, so its bounds are shorter.
// Measured on a server, requests of 17^3 nodes and 5 steps, one at a time,
// beside four of 97^3 (mixed): median latency 29.0 ms with 4 steps and no time
// bound, 11.1 ms with 4 steps and 2 ms, 8.7 ms with 16 steps and 2 ms, 15.3 ms
// with 3 ms for the large and 1 ms for the small; the four took 505, 546, 561
// and 530 ms, ten mixed requests without a steady load 71, 73, 75 and 72 ms.
struct ResBounds {
  int steps;
  double ms;
};
constexpr ResBounds kResRun{128, 100.0}, kResServe{4, 2.0};

// What a step reports.
struct ResStep {
  int32_t iters, sweeps;
  double delta, delta_b, tol;
};

// The kernels: FP64 iterations with the Jacobi or the Chebyshev
// preconditioner, and the mixed form.
enum ResForm { RES_F64, RES_MIXED, RES_CHEB };

// Exchange vectors of the Chebyshev chain (the handle's four chain vectors):
// one per step, so degrees up to 5 run resident.
constexpr int kResChain = 4;

enum ResState : int32_t { RES_ABSENT = 0, RES_RAN = 1, RES_LATE = 2, RES_LOST = 3 };

// What a launch reports per simulation.
struct ResOut {
  int32_t state;   // RES_ABSENT: not every block was resident in time, nothing was done; RES_LATE: the launch's
                   // time was over before the simulation's turn, nothing was done
  int32_t steps;   // steps completed
  int32_t status;  // 0 or kStatusBreakdown (in the step after the completed ones)
  int32_t pad;
  uint64_t samples[3];  // timed direction gathers, updates and replacements
  uint64_t ticks[3];    // and their summed durations (device clock ticks)
  uint64_t count[2];    // iterations and replacements so far (for the next launch)
};

// One simulation of a launch.
struct ResSim {
  Geom g;
  ResShape s;
  const double *rhoc64, *k64;
  const float *rhoc32, *k32;
  double sa64, sbA64, sbL64, Mc64[8], Kc64[8];
  float sa32, sbA32, Mc32[8], Kc32[8];
  const double *F, *pinv64, *lift;
  const float* pinv32;
  double* b;
  double* T[3];    // T^{n-1}, T^{n-2} and a third buffer, rotated from step to step
  void* E[3];      // exchanged P^-1 r (the iterations' precision), used in turn
  void* EX;        // exchanged iterate of a replacement (the iterations' precision)
  double* EX64;    // mixed form: exchanged FP64 iterate of a correction
  double* EC[kResChain];  // exchanged vectors of the Chebyshev chain, one per step
  double ch_inv_c, ch_a[kResChain], ch_b[kResChain];
  void* stash;     // the direction's halo during a replacement: kResHalo values per thread
  unsigned long long* slots;  // 2 sets x kResRep x nblk partials of two words
  unsigned long long* ctl;    // [0] rendezvous, [1] lost
  unsigned long long* launch; // of the launch: [0] simulations that have met and not ended, [1] its start (device clock)
  const double* fs;           // dt * s_n of the launch's steps
  ResStep* rec;               // of the launch's steps
  const double* xyz;
  double* traces;             // of the launch's steps
  ResOut* out;
  double rtol2, inner_rtol;
  uint32_t spin_meet, spin;   // polls before a wait gives up
  int32_t nsens, nsteps, max_iter, stop_rule, R, guess_prev, max_refine, timing, chain;
  // (last: ahead of the vectors these moved the kernels' scalar loads, 1.5% on a 201 x 201 x 26 mixed run)
  int32_t queued;             // not the first simulation of its pass (which always runs)
  uint64_t hold;              // device clock ticks that the launch lasts at most
  int32_t prepared;           // its vectors and slots are as resident_reset_kernel left them
};

// 8-byte words of a simulation's own scratch: the control words (in a cache
// line of their own), the slots of the sums, the stash.  They lie in the fourth
// field buffer, which this form does not use, wherever they fit (most cuts with
// bricks of 9 planes, as batch members have), else in a buffer of their own.
// (A buffer of its own for every simulation, 1.2 MB at 61^3 nodes, 5 MB at
// 101^3, took a batch of 40 simulations of 61^3 nodes from 218 to 240 ms; this
// way 196.)
constexpr size_t kResCtl = 16;
__host__ __device__ constexpr size_t res_slot_words(const ResShape& s) { return (size_t)2 * kResRep * s.nblk * 2; }
__host__ __device__ constexpr size_t res_words(const ResShape& s) {
  return kResCtl + res_slot_words(s) + (size_t)s.nblk * (size_t)s.nthreads * kResHalo;
}

// Values of a brick's node array: its columns with the halo, and one column
// that takes the writes of lanes without a node; a multiple of 4 (alignment).
__host__ __device__ constexpr int res_nodes(int a, int b, int c) { return (((a + 2) * (b + 2) + 1) * (c + 2) + 3) / 4 * 4; }
__host__ __device__ constexpr size_t res_lds(int a, int b, int c, size_t w) {
  return w * ((size_t)res_nodes(a, b, c) + 2 * (size_t)(a + 1) * (b + 1) * (c + 2));
}
// (the Chebyshev chain's vector is a second node array behind these)
__host__ __device__ constexpr size_t res_lds(int a, int b, int c, ResForm f) {
  return res_lds(a, b, c, sizeof(double)) + (f == RES_CHEB ? sizeof(double) * (size_t)res_nodes(a, b, c) : 0);
}

}  // namespace femheat
