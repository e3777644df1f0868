// Whole time steps of a simulation in one kernel (gfx950): the grid is cut
// into bricks, one per block, that stay on chip from step to step.
//
// The two-kernel form streams every vector of Algorithm 1 through HBM (or
// the Infinity Cache) and pays two launches per iteration.  A CU holds
// 160 KB of LDS and 512 KB of registers, so a grid of up to about 1.1M nodes
// fits on the chip: each block keeps, for its brick of a x b x c nodes, the
// search direction with a one-node halo and the element coefficients in LDS
// and r, x and P^-1 in registers, and runs the right-hand side, the initial
// residual, the iterations of Algorithm 1 and (mixed form) the refinement
// sweeps of step after step without leaving the kernel.  What crosses blocks
// is, per iteration, two sums and one layer of P^-1 r around each brick.
//
// What bounds it: at 1M nodes (252 bricks of 34 x 15 x 9) 4.5 us of an
// iteration are the operator's march through LDS (FP64 issue, two waves per
// SIMD), 2.3 us each of the two sums, and the rest the vector updates and the
// exchange between them; at 5k nodes (18 bricks) the march takes 1.0 us and a
// sum 1.3 us, most of it the way of a word from one XCD to the others and
// back.  Measured per iteration, two-kernel form -> this form (runs of 20-40
// steps): 101^3 FP64 28.6 -> 13.5 us, mixed 22.8 -> 12.5 us; 201 x 201 x 26
// mixed 21.4 -> 10.0 us; 49^3 FP64 11.8 -> 5.9 us; 17^3 FP64 16.3 -> 5.8 us.
//
// The arithmetic at a node is that of the two-kernel form, operation by
// operation (layer_contributions, and the updates below); only the dot
// products are summed in another grouping (per brick).
//
// With the Chebyshev preconditioner P^-1 r is a chain of m - 1 operator
// applications: its vector takes a second node array in LDS, its residual and
// sum take registers, and each step is a march and an exchange of the brick's
// surface without a sum (at 65^3 nodes and m = 3: 45 -> 18.0 us per iteration,
// four kernels' launches and passes over memory before).
//
// Crossing blocks.  Other XCDs' L2s do not see plain stores, so everything
// that crosses goes through device-scope atomics (loads and stores past the
// L2s), and no fence is needed:
//  * a sum: each block stores its partial as two 8-byte words tagged with the
//    sum's number, in kResRep copies (so that not every block polls the same
//    lines), and every block polls all partials until their tags match and
//    adds them in one fixed order: every block holds the same value.  Passing
//    a sum also means that every block has reached it.  Two sets of slots
//    alternate: a block stores into a set again only after it has passed the
//    next sum, which every block reaches only after reading this one.
//  * a halo: each block stores its brick's surface into a node vector that
//    holds a marker (a signalling NaN, which no operation returns) where
//    nothing has been stored; the neighbours poll their halo nodes until none
//    holds the marker.  No barrier is needed, so the exchange overlaps the
//    sum after it.  The owner puts the marker back once a later sum has shown
//    that everybody has read; it waits for these stores before it publishes
//    the next sum that is not an exchange itself, and at least one such sum
//    lies before the vector's next use.  (A vector of the chain is used once
//    per iteration and cleared behind the iteration's second sum.)
//
// Every block of the simulation has to be resident for that.  A launch first
// meets (rendezvous): blocks count in at one word and wait until all have; a
// block whose wait runs out marks the word, which succeeds only while the
// count is incomplete, and then no block proceeds.  Nothing has been written
// by then, so the host takes the two-kernel form.  (A block that comes after
// the launch's time is over does not count in, and marks the word too: the
// simulation waits for the next launch.)  The blocks of a launch may
// outnumber the compute units: those of a later simulation then wait for an
// earlier one to end, and the time that one runs does not count.  (It ends by
// itself.  With a long bound instead, two processes whose launches each held
// part of the device stood still for all of it.)  After the meeting every wait
// is for a block that runs, and the bound on it only guards against the
// impossible.
#pragma once

#include <utility>

#include "gather.hpp"
#include "resident_types.hpp"
#include "vector_kernels.hpp"

namespace femheat {

constexpr unsigned long long kResAbort = 1ull << 63;

template <typename V>
struct ResWord;
template <>
struct ResWord<double> {
  using U = unsigned long long;
  static constexpr U kEmpty = 0xFFF7DEADBEEF0001ull;
};
template <>
struct ResWord<float> {
  using U = unsigned int;
  static constexpr U kEmpty = 0xFFB7DEADu;
};

#if defined(__HIP_DEVICE_COMPILE__)
template <typename U>
__device__ __forceinline__ U dev_ld(const U* base, uint32_t i) {
  gcptr<char> b = (gcptr<char>)base;
  return __hip_atomic_load((gcptr<U>)(b + (uint32_t)(i * (uint32_t)sizeof(U))), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename U>
__device__ __forceinline__ void dev_st(U* base, uint32_t i, U v) {
  gptr<char> b = (gptr<char>)base;
  __hip_atomic_store((gptr<U>)(b + (uint32_t)(i * (uint32_t)sizeof(U))), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// base[i] += v; what it becomes
template <typename U>
__device__ __forceinline__ U dev_add(U* base, uint32_t i, U v) {
  gptr<char> b = (gptr<char>)base;
  return __hip_atomic_fetch_add((gptr<U>)(b + (uint32_t)(i * (uint32_t)sizeof(U))), v, __ATOMIC_RELAXED,
                                __HIP_MEMORY_SCOPE_AGENT) + v;
}
#else
template <typename U>
__device__ U dev_add(U* base, uint32_t i, U v) {
  return base[i] += v;
}
template <typename U>
__device__ U dev_ld(const U* base, uint32_t i) {
  return base[i];
}
template <typename U>
__device__ void dev_st(U* base, uint32_t i, U v) {
  base[i] = v;
}
#endif

// (lambdas are inlined first of all, so that the arrays they refer to can be split)
#define FEM_INLINE __attribute__((always_inline))

// f(0), f(1), ... f(N - 1), each with a constant: an array that is only
// indexed through it is split into registers before the loops around it are
// looked at (indexed by a loop to be unrolled later, it becomes one long
// vector register, and those spill).
template <class F, int... I>
__device__ __forceinline__ void each_of(F& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void each(F f) {
  each_of(f, std::make_integer_sequence<int, N>{});
}

template <typename V>
__device__ __forceinline__ typename ResWord<V>::U to_word(V v) {
  typename ResWord<V>::U u;
  __builtin_memcpy(&u, &v, sizeof(V));
  return u == ResWord<V>::kEmpty ? (u | (sizeof(V) == 8 ? (typename ResWord<V>::U)1 << (8 * sizeof(V) - 13)
                                                        : (typename ResWord<V>::U)1 << 22))
                                 : u;
}
template <typename V>
__device__ __forceinline__ V from_word(typename ResWord<V>::U u) {
  V v;
  __builtin_memcpy(&v, &u, sizeof(V));
  return v;
}

// The same value in every lane, known to the compiler as such: what a block
// decides on (sums, flags) comes out of LDS, and branches on it would
// otherwise be compiled per lane, with the loop's scalars in vector registers.
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ float uniform(float v) { return __int_as_float(uniform(__float_as_int(v))); }
__device__ __forceinline__ double uniform(double v) {
  int w[2];
  __builtin_memcpy(w, &v, 8);
  w[0] = uniform(w[0]);
  w[1] = uniform(w[1]);
  __builtin_memcpy(&v, w, 8);
  return v;
}

// Sum over a wave, the same value in every lane: within rows of 16 lanes by
// cross-lane operands of the adds (two exchanges in a quad, two mirrors),
// the four rows through scalar registers.  (A butterfly of six shuffles goes
// through LDS each time: 0.3 us longer, four times an iteration.)
template <int kCtrl>
__device__ __forceinline__ double row_add(double v) {
  int w[2], x[2];
  __builtin_memcpy(w, &v, 8);
  x[0] = __builtin_amdgcn_update_dpp(0, w[0], kCtrl, 0xf, 0xf, false);
  x[1] = __builtin_amdgcn_update_dpp(0, w[1], kCtrl, 0xf, 0xf, false);
  double o;
  __builtin_memcpy(&o, x, 8);
  return v + o;
}
__device__ __forceinline__ double lane_value(double v, int lane) {
  int w[2];
  __builtin_memcpy(w, &v, 8);
  w[0] = __builtin_amdgcn_readlane(w[0], lane);
  w[1] = __builtin_amdgcn_readlane(w[1], lane);
  __builtin_memcpy(&v, w, 8);
  return v;
}
__device__ __forceinline__ double wave_sum(double v) {
  v = row_add<0xB1>(v);   // quad_perm 1, 0, 3, 2
  v = row_add<0x4E>(v);   // quad_perm 2, 3, 0, 1
  v = row_add<0x141>(v);  // row_half_mirror
  v = row_add<0x140>(v);  // row_mirror
  return ((lane_value(v, 0) + lane_value(v, 16)) + lane_value(v, 32)) + lane_value(v, 48);
}

// The value v, opaque to the compiler: addresses formed from it are formed
// where they are used.  (Hoisted out of the kernel's loops, the addresses
// of all its phases would take the registers that the brick's vectors need.)
__device__ __forceinline__ int here(int v) {
  asm volatile("" : "+v"(v));
  return v;
}
__device__ __forceinline__ uint32_t here(uint32_t v) {
  asm volatile("" : "+v"(v));
  return v;
}
__device__ __forceinline__ double here(double v) {
  asm volatile("" : "+v"(v));
  return v;
}
__device__ __forceinline__ float here(float v) {
  asm volatile("" : "+v"(v));
  return v;
}

// LDS layout of a brick.  Along z a column of nodes (or of elements) is
// contiguous, L + 2 values (or pairs rho*c, k) apart from its x-neighbour: the
// planes of a march are immediate offsets from three row addresses, and L is
// odd, so the lanes of a wave, one column each, read distinct banks (8-byte
// reads L + 2 apart for nodes, 16-byte reads L + 2 apart for coefficients).
// (Planes x-fastest, as the two-kernel gather stages them, cost an address
// register per plane and row, and the register arrays below then spill.)
template <int L>
constexpr int kResPitch = L + 2;

// A block's brick, its thread's column and the thread's share of the halo.
// Lanes without a node (idle lanes, columns past the grid) and planes past the
// grid carry P^-1 = 0 and zeros throughout, and unused halo entries the value
// 0 and the spare column, so that none of the vector updates needs a test.
// (A brick with fewer than L planes ends at the grid's last plane: the planes
// above are outside, where the halo's value is 0 as well.)
struct Brick {
  int nz;                     // planes of this brick (<= c)
  int pw, cw;                 // columns per row of the node and element arrays
  int rd, wr;                 // LDS index of the column's (-x, -y) neighbour, plane 0; of its own plane 0
  int cf;                     // of its (-x, -y) element column
  bool ok;                    // the thread has a column in the grid
  uint32_t smask;             // bit z: the column's plane z is on the brick's surface
  uint32_t i0, ps;            // node of the column's first plane; nodes per plane
  uint32_t hmask;             // bit k: halo entry k is a node of another brick
  int hidx[kResHalo];         // LDS index of halo entry k
  uint32_t hnode[kResHalo];   // its node
};

template <int L>
__device__ inline void brick_setup(Brick& B, const Geom& g, const ResShape& s, uint32_t blk, int& x0, int& y0, int& z0) {
  constexpr int P = kResPitch<L>;
  const int t = threadIdx.x, nt = s.nthreads;
  const int bx = (int)(blk % (uint32_t)s.nbx), by = (int)(blk / (uint32_t)s.nbx % (uint32_t)s.nby),
            bz = (int)(blk / ((uint32_t)s.nbx * (uint32_t)s.nby));
  x0 = bx * s.a;
  y0 = by * s.b;
  z0 = bz * L;
  const int na = min(s.a, g.px - x0), nb = min(s.b, g.py - y0);
  B.nz = min(L, g.pz - z0);
  B.pw = s.a + 2;
  B.cw = s.a + 1;
  const int pcols = B.pw * (s.b + 2), spare = pcols * P;
  const bool has = t < s.a * s.b;
  const int ltx = has ? t % s.a : 0, lty = has ? t / s.a : 0;
  B.ok = has && ltx < na && lty < nb;
  const bool side = ltx == 0 || ltx == na - 1 || lty == 0 || lty == nb - 1;
  B.smask = (!B.ok || s.nblk == 1) ? 0u : side ? (1u << B.nz) - 1u : (1u | (1u << (B.nz - 1)));
  B.rd = (lty * B.pw + ltx) * P;
  B.wr = has ? B.rd + (B.pw + 1) * P : spare;
  B.cf = (lty * B.cw + ltx) * 2 * P;
  B.ps = (uint32_t)g.px * (uint32_t)g.py;
  B.i0 = (B.ok ? (uint32_t)(x0 + ltx) + (uint32_t)g.px * (uint32_t)(y0 + lty) : 0u) + B.ps * (uint32_t)z0;
  // halo nodes: the planes below and above, then a ring around each plane
  const int ring = 2 * B.pw + 2 * s.b, total = 2 * pcols + L * ring;
  B.hmask = 0;
  each<kResHalo>([&](auto k) FEM_INLINE {
    const int h = t + k * nt;
    B.hidx[k] = spare;
    B.hnode[k] = 0;
    if (h < total) {
      int lx, ly, lz;
      if (h < 2 * pcols) {
        lz = h < pcols ? 0 : L + 1;
        const int o = h < pcols ? h : h - pcols;
        ly = o / B.pw;
        lx = o - ly * B.pw;
      } else {
        int o = h - 2 * pcols;
        lz = 1 + o / ring;
        o %= ring;
        if (o < 2 * B.pw) {
          ly = o < B.pw ? 0 : s.b + 1;
          lx = o < B.pw ? o : o - B.pw;
        } else {
          o -= 2 * B.pw;
          ly = 1 + (o >> 1);
          lx = (o & 1) ? s.a + 1 : 0;
        }
      }
      B.hidx[k] = (ly * B.pw + lx) * P + lz;
      const int x = x0 - 1 + lx, y = y0 - 1 + ly, z = z0 - 1 + lz;
      if (x >= 0 && x < g.px && y >= 0 && y < g.py && z >= 0 && z < g.pz) {
        B.hmask |= 1u << k;
        B.hnode[k] = (uint32_t)x + (uint32_t)g.px * (uint32_t)y + B.ps * (uint32_t)z;
      }
    }
  });
}

// The operator at the nodes of the thread's column: acc[z] for plane z of
// the brick, from the input in D (planes 0 .. L+1) and the coefficients in C
// (layers 0 .. L).  Straight-line code.  The next plane and the next layer's
// coefficients are read while a layer is summed.
template <typename V, int KIND, int L>
__device__ __forceinline__ void brick_apply(const Brick& B, const V* D, const V* C, const V* Mc, const V* Kc,
                                            V (&acc)[L]) {
  constexpr int P = kResPitch<L>;
  const int rd = here(B.rd), cf = here(B.cf);
  const V* row[3] = {D + rd, D + rd + B.pw * P, D + rd + 2 * B.pw * P};
  const V* crow[2] = {C + cf, C + cf + B.cw * 2 * P};
  auto plane = [&](auto k, PlaneQ<V>& q) FEM_INLINE {
    q.b[0] = row[0][k];
    q.ym = row[0][P + k];
    q.b[1] = row[0][2 * P + k];
    q.xm = row[1][k];
    q.c = row[1][P + k];
    q.xp = row[1][2 * P + k];
    q.b[2] = row[2][k];
    q.yp = row[2][P + k];
    q.b[3] = row[2][2 * P + k];
  };
  using V2 = std::conditional_t<sizeof(V) == 8, double2, float2>;
  struct Coefs {
    V a[4], b[4];
  };
  auto coefs = [&](auto k, Coefs& c) FEM_INLINE {
    each<4>([&](auto e) FEM_INLINE {
      constexpr int sx = e & 1, sy = e >> 1;
      const V2 w = *reinterpret_cast<const V2*>(crow[sy] + sx * 2 * P + 2 * k);  // one aligned read
      c.a[e] = w.x;
      c.b[e] = w.y;
    });
  };
  PlaneQ<V> lo, hi, next;
  Coefs cc, cn;
  plane(std::integral_constant<int, 0>{}, lo);
  plane(std::integral_constant<int, 1>{}, hi);
  coefs(std::integral_constant<int, 0>{}, cc);
  V carry = V(0);
  each<L + 1>([&](auto k) FEM_INLINE {
    // one layer at a time: the compiler would otherwise read the whole column
    // into registers first, which the brick's vectors need, and form the sums
    // where they are used
    if constexpr (k < L) {
      plane(std::integral_constant<int, k + 2>{}, next);
      coefs(std::integral_constant<int, k + 1>{}, cn);
    }
    __builtin_amdgcn_sched_barrier(0);
    V p_lo, p_hi;
    auto coef = [&](int sx, int sy, V& a, V& bk) FEM_INLINE {
      a = cc.a[sy * 2 + sx];
      bk = cc.b[sy * 2 + sx];
    };
    layer_contributions<V, KIND>(lo, hi, false, coef, Mc, Kc, p_lo, p_hi);
    if constexpr (k > 0) acc[k - 1] = carry + p_lo;
    carry = p_hi;
    lo = hi;
    hi = next;
    cc = cn;
    if constexpr (k > 0) asm volatile("" : "+v"(acc[k - 1]), "+v"(carry)::"memory");
    __builtin_amdgcn_sched_barrier(0);
  });
}

// Sum of N values in LDS (all read at once).
template <int N>
__device__ __forceinline__ double sum_of(const double* v) {
  if constexpr (N == 1)
    return v[0];
  else
    return sum_of<N / 2>(v) + sum_of<N / 2>(v + N / 2);
}

// The blocks of one simulation.
struct Meet {
  unsigned long long* slots;
  unsigned long long* ctl;
  uint32_t G, blk, seq, spin;
  int nt;  // threads that work (waves past them have left)
};

// Wave sums of a block, zero for waves that have left (two sets alternate),
// and the waves' shares of the partials.
struct MeetLds {
  double own[2][kResThreads / 64], all[kResThreads / 64];
};

// Sum of v over every thread of every block, the same value in all of them,
// or anything with *lost set.  kHalo: also reads the thread's halo nodes of E
// (published by their owners before their own call) into hv (0 where there is
// none).  kWait: earlier stores of the block complete before its partial is
// published.  gap(): work to do while the partials travel.
//
// Each wave polls a share of the partials, and the block adds the shares: every
// wave polling all of them saved a barrier and a pass through LDS but added
// polls, which slow each other down (37^3 nodes 5.85 against 5.45 us per
// iteration, 25^3 5.10 against 4.90, 17^3 and below equal within 1%).
template <bool kWait, typename V, bool kHalo, class Gap>
__device__ __forceinline__ double meet_sum(Meet& M, MeetLds& lds, double v, const typename ResWord<V>::U* E,
                                           const Brick& B, V (&hv)[kResHalo], int* lost, Gap gap) {
  constexpr int kW = kResThreads / 64;
  const int t = here((int)threadIdx.x), lane = t & 63, wid = t >> 6;
  v = wave_sum(v);
  const uint32_t seq = ++M.seq;
  if (kWait) __builtin_amdgcn_s_waitcnt(0);
  if (lane == 0) lds.own[seq & 1][wid] = v;
  __syncthreads();
  const double own = sum_of<kW>(lds.own[seq & 1]);
  if (kHalo) each<kResHalo>([&](auto k) FEM_INLINE { hv[k] = V(0); });
  if (M.G == 1) return uniform(own);  // no halo either: the brick is the grid
  unsigned long long* set = M.slots + (size_t)(seq & 1) * kResRep * M.G * 2;
  if (t < 2 * kResRep) {
    unsigned long long u;
    __builtin_memcpy(&u, &own, 8);
    const unsigned long long half = (t & 1) ? (u & 0xffffffffull) : (u >> 32);
    dev_st(set, ((uint32_t)(t >> 1) * M.G + M.blk) * 2 + (uint32_t)(t & 1), ((unsigned long long)seq << 32) | half);
  }
  gap();
  const unsigned long long* mine = set + (size_t)(M.blk % kResRep) * M.G * 2;
  constexpr int kS = 4;  // partials per thread at most: kResBlocks / 64
  using U = typename ResWord<V>::U;
  // Every round reads the partials again (what has arrived stays), and the
  // halo until the wave has all of it: the rounds after that are shorter and
  // leave the fabric to those who still wait (49^3 6.36 -> 5.88 us per
  // iteration, 101^3 13.9 -> 13.5; entry by entry, with a branch for each,
  // 6.07 and 13.6, and a pause between rounds lost more than it gave).
  const uint32_t first = (uint32_t)t, step = (uint32_t)M.nt;
  double part[kS] = {0.0, 0.0, 0.0, 0.0};
  bool open = kHalo;  // some lane of the wave waits for its halo
  for (uint32_t it = 0;; ++it) {
    unsigned long long wa[kS], wb[kS];
    U h[kResHalo];
    if (open) each<kResHalo>([&](auto k) FEM_INLINE { h[k] = dev_ld(E, here(B.hnode[k])); });
    bool there = true;
    each<kS>([&](auto k) FEM_INLINE {
      if (k * step < M.G) {  // uniform
        const uint32_t s = first + k * step;
        if (s < M.G) {
          wa[k] = dev_ld(mine, s * 2);
          wb[k] = dev_ld(mine, s * 2 + 1);
        }
      }
    });
    each<kS>([&](auto k) FEM_INLINE {
      if (k * step < M.G) {
        if (first + k * step < M.G) {
          there = there && (uint32_t)(wa[k] >> 32) == seq && (uint32_t)(wb[k] >> 32) == seq;
          const unsigned long long u = (wa[k] << 32) | (wb[k] & 0xffffffffull);
          __builtin_memcpy(&part[k], &u, 8);
        }
      }
    });
    if (open) {
      bool halo = true;
      each<kResHalo>([&](auto k) FEM_INLINE {
        const bool mine_k = (B.hmask >> k) & 1u;
        halo = halo && (!mine_k || h[k] != ResWord<V>::kEmpty);
        hv[k] = mine_k ? from_word<V>(h[k]) : V(0);
      });
      open = __builtin_amdgcn_ballot_w64(!halo) != 0;
    }
    if (!open && __builtin_amdgcn_ballot_w64(!there) == 0) break;
    if (it >= M.spin || ((it & 4095u) == 4095u && dev_ld(M.ctl, 1) != 0)) {
      *lost = 1;
      break;
    }
  }
  const double x = wave_sum(((part[0] + part[1]) + part[2]) + part[3]);
  if (lane == 0) lds.all[wid] = x;
  __syncthreads();
  return uniform(sum_of<kW>(lds.all));
}

// Reads the thread's halo nodes of E into hv (no sum).
template <typename V>
__device__ __forceinline__ void meet_halo(const Meet& M, const typename ResWord<V>::U* E, const Brick& B,
                                          V (&hv)[kResHalo], int* lost) {
  using U = typename ResWord<V>::U;
  for (uint32_t it = 0;; ++it) {
    U h[kResHalo];
    each<kResHalo>([&](auto k) FEM_INLINE { h[k] = dev_ld(E, here(B.hnode[k])); });
    bool there = true;
    each<kResHalo>([&](auto k) FEM_INLINE {
      const bool mine = (B.hmask >> k) & 1u;
      there = there && (!mine || h[k] != ResWord<V>::kEmpty);
      hv[k] = mine ? from_word<V>(h[k]) : V(0);
    });
    if (M.G == 1 || __builtin_amdgcn_ballot_w64(!there) == 0) break;
    if (it >= M.spin || ((it & 4095u) == 4095u && dev_ld(M.ctl, 1) != 0)) {
      *lost = 1;
      break;
    }
  }
}

// The column's surface nodes of a brick: f(z, node) for every plane z whose
// node another brick has in its halo (or might have).
template <int L, class F>
__device__ __forceinline__ void on_surface(const Brick& B, F f) {
  const uint32_t i0 = here(B.i0), m = here(B.smask);
  each<L>([&](auto z) FEM_INLINE {
    if ((m >> z) & 1u) f(z, i0 + B.ps * (uint32_t)z);
  });
}
template <typename V, int L>
__device__ __forceinline__ void clear_surface(const Brick& B, typename ResWord<V>::U* E) {
  on_surface<L>(B, [&](auto, uint32_t i) FEM_INLINE { dev_st(E, i, ResWord<V>::kEmpty); });
}

// Scaled coefficients of the brick's layers into C (0 outside the grid);
// kRho: rho*c too, else k only (another operator of the same precision).
template <typename V, int L, bool kRho>
__device__ inline void fill_coefficients(const Brick& B, const Geom& g, const ResShape& s, int x0, int y0, int z0,
                                         const V* rhoc, const V* kc, V sa, V sb, V* C) {
  const int cs = B.cw * (s.b + 1);
  const uint32_t ls = (uint32_t)g.nx * (uint32_t)g.ny;
  // a column of elements per thread and round
  for (int o = here((int)threadIdx.x); o < cs; o += s.nthreads) {
    const int cy = o / B.cw, cx = o - cy * B.cw;
    const int ex = x0 - 1 + cx, ey = y0 - 1 + cy;
    const bool in = ex >= 0 && ex < g.nx && ey >= 0 && ey < g.ny;
    const uint32_t e0 = in ? (uint32_t)ex + (uint32_t)g.nx * (uint32_t)ey : 0u;
    V* const p = C + o * kResPitch<L> * 2;
    constexpr int kChunk = L == 9 ? 5 : L + 1;  // layers read at once (registers)
    each<(L + 1) / kChunk>([&](auto q) FEM_INLINE {
      V kk[kChunk], rr[kChunk];
      __builtin_amdgcn_sched_barrier(0);
      each<kChunk>([&](auto c) FEM_INLINE {
        const int ez = z0 - 1 + q * kChunk + c;  // (the same in every lane)
        const uint32_t e = e0 + ls * (uint32_t)min(max(ez, 0), g.nz - 1);
        kk[c] = gld(kc, e);
        if constexpr (kRho) rr[c] = gld(rhoc, e);
      });
      each<kChunk>([&](auto c) FEM_INLINE {
        constexpr int l = q * kChunk + c;
        const int ez = z0 - 1 + l;
        const bool inside = in && ez >= 0 && ez < g.nz;
        if constexpr (kRho) p[2 * l] = inside ? sa * rr[c] : V(0);
        p[2 * l + 1] = inside ? sb * kk[c] : V(0);
      });
    });
  }
}

// In-kernel samples of the phases (FEM_TIMING): one iteration in
// kResSampleEvery and one replacement in kResReplaceEvery.
constexpr uint64_t kResSampleEvery = 64, kResReplaceEvery = 8;
struct ResClock {
  uint64_t t0, t1;
  int32_t pick, pick_rep;  // this iteration, this replacement is in the sample
  // by the lead thread of the simulation; the other threads pass
  __device__ void direction(bool lead, ResOut* o) {
    if (!lead) return;
    pick = o->count[0]++ % kResSampleEvery == 0;
    pick_rep = 0;
    t0 = wall_clock64();
  }
  __device__ void summed(bool lead, ResOut* o) {
    if (!lead) return;
    t1 = wall_clock64();
    if (pick) {
      o->samples[0] += 1;
      o->ticks[0] += t1 - t0;
    }
  }
  __device__ void replacement(bool lead, ResOut* o) {
    if (lead) pick_rep = o->count[1]++ % kResReplaceEvery == 0;
  }
  __device__ void updated(bool lead, ResOut* o, bool replaced) {
    if (!lead || !(replaced ? pick_rep : pick)) return;
    o->samples[replaced ? 2 : 1] += 1;
    o->ticks[replaced ? 2 : 1] += wall_clock64() - t1;
  }
};

// Puts the marker into the exchange vectors of every simulation of a launch
// and clears its slots and words; the launch's own words count from here.
[[maybe_unused]] static __global__ void __launch_bounds__(256) resident_reset_kernel(const ResSim* sims, uint32_t nsims,
                                                                                    int mixed) {
  const uint32_t tid = blockIdx.x * blockDim.x + threadIdx.x, n = gridDim.x * blockDim.x;
  if (blockIdx.y == 0 && tid == 0) {
    gst(sims->launch, 0u, 0ull);
    gst(sims->launch, 1u, (unsigned long long)wall_clock64());
  }
  for (uint32_t k = blockIdx.y; k < nsims; k += gridDim.y) {
    const ResSim& S = sims[k];
    const uint32_t N = S.g.N;
    if (tid < 2) gst(S.ctl, tid, 0ull);
    // (a simulation whose turn did not come in the last launch left all but its
    // words alone: clearing its vectors again in every launch until it comes
    // took a server of 48 mixed requests of 98^3 nodes 968 ms instead of 903)
    if (S.s.nblk == 1 || S.prepared) continue;
    for (uint32_t i = tid; i < N; i += n) {
      if (mixed) {
        for (void* E : S.E) gst(static_cast<unsigned int*>(E), i, ResWord<float>::kEmpty);
        gst(static_cast<unsigned int*>(S.EX), i, ResWord<float>::kEmpty);
        gst(reinterpret_cast<unsigned long long*>(S.EX64), i, ResWord<double>::kEmpty);
      } else {
        for (void* E : S.E) gst(static_cast<unsigned long long*>(E), i, ResWord<double>::kEmpty);
        gst(static_cast<unsigned long long*>(S.EX), i, ResWord<double>::kEmpty);
        for (int c = 0; c < S.chain; ++c) gst(reinterpret_cast<unsigned long long*>(S.EC[c]), i, ResWord<double>::kEmpty);
      }
    }
    for (uint32_t i = tid; i < 2u * kResRep * S.s.nblk * 2u; i += n) gst(S.slots, i, 0ull);
  }
}

// Steps of one simulation by its blocks.  V: precision of the iterations
// (double: the FP64 form; float: the mixed form's inner solves); L: planes
// of a brick; CHEB: P^-1 stands for the Chebyshev preconditioner, a chain of
// operator applications (FP64); table: block -> (simulation, its brick),
// nullptr: one simulation.
template <typename V, int KIND, int L, bool CHEB>
__global__ void __launch_bounds__(kResThreads) resident_kernel(const ResSim* __restrict__ sims,
                                                               const uint2* __restrict__ table) {
  constexpr bool kMixed = sizeof(V) == 4;
  extern __shared__ __align__(16) unsigned char res_smem[];
  __shared__ int lost, go;
  __shared__ ResClock clk;
  __shared__ uint64_t until;  // (of the lead block) the device clock at which the launch is to end
  __shared__ __align__(16) MeetLds mlds;
  uint32_t sim = 0, blk = blockIdx.x;
  if (table) {
    const uint2 w = table[blockIdx.x];
    sim = (uint32_t)__builtin_amdgcn_readfirstlane((int)w.x);
    blk = (uint32_t)__builtin_amdgcn_readfirstlane((int)w.y);
  }
  const ResSim& S = sims[sim];
  const Geom& g = S.g;
  if ((int)threadIdx.x >= S.s.nthreads) return;  // whole waves: the launch's widest brick sets the block
  Meet M{S.slots, S.ctl, S.s.nblk, blk, 0u, S.spin, S.s.nthreads};
  if (threadIdx.x < kResThreads / 64) mlds.own[0][threadIdx.x] = mlds.own[1][threadIdx.x] = mlds.all[threadIdx.x] = 0.0;
  if (threadIdx.x == 0) {
    lost = 0;
    go = 1;
    bool all = M.G == 1;  // this block completes the meeting
    until = gld(S.launch, 1u) + S.hold;
    const bool late = S.queued && wall_clock64() > until;  // no turn in this launch
    if (late) S.out->state = RES_LATE;
    if (M.G > 1) {
      __attribute__((address_space(1))) unsigned long long* w =
          (__attribute__((address_space(1))) unsigned long long*)S.ctl;
      const uint32_t limit = late ? 0u : S.spin_meet;
      // (a limit of no polls fails every meeting: no block counts in.  Counting
      // in first, all blocks often had before any of them gave up.)
      unsigned long long now = limit == 0 ? dev_ld(S.ctl, 0) : dev_add(S.ctl, 0, 1ull);
      all = now == M.G;
      for (uint32_t it = 0; !(now & kResAbort) && now < M.G; ++it) {
        if ((it & 63u) == 63u && dev_ld(S.launch, 0) != 0) it = 0;
        if (it >= limit) {
          unsigned long long want = now;
          if (__hip_atomic_compare_exchange_strong(w, &want, now | kResAbort, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT))
            now |= kResAbort;
          else
            now = want;
        } else {
          now = dev_ld(S.ctl, 0);
        }
      }
      if (now & kResAbort) go = 0;
    } else if (late) {
      go = 0;
      all = false;
    }
    if (all) (void)dev_add(S.launch, 0, 1ull);
  }
  __syncthreads();
  if (!uniform(go)) return;

  Brick B;
  int x0, y0, z0;
  brick_setup<L>(B, g, S.s, blk, x0, y0, z0);
  const int nodes = res_nodes(S.s.a, S.s.b, L);
  double* const D64 = reinterpret_cast<double*>(res_smem);
  double* const C64 = D64 + nodes;
  V* const D = reinterpret_cast<V*>(res_smem);
  V* const C = D + nodes;
  const int chain_at = CHEB ? nodes + 2 * (S.s.a + 1) * (S.s.b + 1) * kResPitch<L> : 0;  // the chain's vector, from D
  // The operator in precision W (general boxes: their 16 weights, read through
  // the scalar cache for each application; held across the loop they crowd the
  // scalar registers and the waits between blocks run through spilled ones).
  auto apply = [&](auto* at, auto* coefs, auto& acc) FEM_INLINE {
    using W = std::remove_reference_t<decltype(*at)>;
    W Mc[8], Kc[8];
    if constexpr (KIND == kElemBox) {
      using K = const __attribute__((address_space(4))) W*;
      const ResSim* from = &S;
      asm volatile("" : "+s"(from));
      K m, k;
      if constexpr (sizeof(W) == 8) {
        m = (K)from->Mc64;
        k = (K)from->Kc64;
      } else {
        m = (K)from->Mc32;
        k = (K)from->Kc32;
      }
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        Mc[c] = m[c];
        Kc[c] = k[c];
      }
    }
    brick_apply<W, KIND, L>(B, at, coefs, Mc, Kc, acc);
  };
  using U = typename ResWord<V>::U;
  using U64 = ResWord<double>::U;
  // the vectors of the exchanges of P^-1 r: the next one's, the one's after
  // it, and the last one's
  U *E0 = static_cast<U*>(S.E[0]), *E1 = static_cast<U*>(S.E[1]), *E2 = static_cast<U*>(S.E[2]);
  U* const EX = static_cast<U*>(S.EX);
  const int nz = B.nz;
  auto column = [&](auto* at) FEM_INLINE { return at + here(B.wr) + 1; };  // the column's own planes in LDS
  // f(z, i): the column's nodes i in the grid (lanes without a node: any node, for values to be dropped)
  auto rows = [&](auto f) FEM_INLINE {
    const uint32_t i0 = here(B.i0);
    each<L>([&](auto z) FEM_INLINE {
      if (z < nz) f(z, i0 + B.ps * (uint32_t)z);
    });
  };
  auto cells = [&](auto f) FEM_INLINE { each<L>(f); };  // f(z): the column's planes
  // f(k, o): halo entry k, at o in a node array in LDS
  auto halo = [&](auto f) FEM_INLINE {
    each<kResHalo>([&](auto k) FEM_INLINE { f(k, here(B.hidx[k])); });
  };
  V p[L], r[L], x[L], q[L], hv[kResHalo];
  double x64[kMixed ? L : 1], r64[kMixed ? L : 1], hd[kResHalo];
  each<L>([&](auto z) FEM_INLINE {
    p[z] = r[z] = x[z] = q[z] = V(0);
    if constexpr (kMixed) x64[z] = r64[z] = 0.0;
  });
  rows([&](auto z, uint32_t i) FEM_INLINE {
    V v;
    if constexpr (kMixed)
      v = gld(S.pinv32, i);
    else
      v = gld(S.pinv64, i);
    p[z] = B.ok ? v : V(0);
  });

  const bool lead = blk == 0 && threadIdx.x == 0;
  const bool timed = S.timing != 0;
  double *T1 = S.T[0], *T2 = S.T[1], *T3 = S.T[2];
  auto dld = [&](const double* v, uint32_t i) FEM_INLINE {
    return from_word<double>(dev_ld(reinterpret_cast<const U64*>(v), i));
  };
  const double rtol2 = S.rtol2;
  const int max_iter = S.max_iter, stop_rule = S.stop_rule, R = S.R;

  // the step and its outer solve
  int m = 0, its = 0, sweeps = 0, status = 0;
  double delta_b = 0.0, odelta = 0.0, odelta0 = 0.0, otol = 0.0;
  // the current solve (the outer one in the FP64 form, an inner one in the mixed form)
  double delta = 0.0, tol = 0.0, rt2 = rtol2;
  V alpha = V(0), beta = V(0);
  int j = 0;
  bool first = true;      // no iteration yet
  bool fresh = false;     // the last exchange may not have been read by all
  U* stale = nullptr;     // one that has, and is to be cleared
  // the Chebyshev chain: its step, what it preconditions, its residual and sum
  int ck = 0, chain_of = 0;
  V cr[CHEB ? L : 1], y[CHEB ? L : 1];

  // T^{n-1} and its halo in D, L's coefficients in C
  auto start_step = [&]() FEM_INLINE {
    if (m == 0 || kMixed)
      fill_coefficients<double, L, true>(B, g, S.s, x0, y0, z0, S.rhoc64, S.k64, S.sa64, S.sbL64, C64);
    else
      fill_coefficients<double, L, false>(B, g, S.s, x0, y0, z0, S.rhoc64, S.k64, S.sa64, S.sbL64, C64);
    double* const own64 = column(D64);
    double v[L], w[kResHalo];
    cells([&](auto z) FEM_INLINE { v[z] = 0.0; });
    rows([&](auto z, uint32_t i) FEM_INLINE { v[z] = dld(T1, i); });
    halo([&](auto k, int) FEM_INLINE { w[k] = ((B.hmask >> k) & 1u) ? dld(T1, B.hnode[k]) : 0.0; });
    cells([&](auto z) FEM_INLINE { own64[z] = B.ok ? v[z] : 0.0; });
    halo([&](auto k, int o) FEM_INLINE { D64[o] = w[k]; });
  };
  // A sum without an exchange: while its partials travel, the exchange before
  // the last one, which every block has read by now, is cleared; the sum shows
  // that every block has read the last one too.  (The clearing stores complete
  // before the next such sum is published, and that one lies before the next
  // use of the vector, two exchanges on.)
  auto plain_sum = [&](double part) FEM_INLINE {
    const double v = meet_sum<true, V, false>(M, mlds, part, nullptr, B, hv, &lost, [&]() FEM_INLINE {
      if (stale) clear_surface<V, L>(B, stale);
    });
    stale = fresh ? E2 : nullptr;
    fresh = false;
    return v;
  };
  auto put = [&](auto* E, auto value) FEM_INLINE {
    using W = decltype(value(std::integral_constant<int, 0>{}));
    on_surface<L>(B, [&](auto z, uint32_t i) FEM_INLINE { dev_st(E, i, to_word<W>(value(z))); });
  };

  // What the brick in D is when the operator is applied to it.
  enum { kRhs, kResidual, kDirection, kReplace, kChain };
  int ph = kRhs;
  // After delta_b: x0 by the guess rule on the brick and its halo, A's coefficients.
  auto start_solve = [&]() FEM_INLINE {
    const bool zero = stop_rule == 0 && delta_b == 0.0;
    double* const own64 = column(D64);
    // (everything is read before it is used: a branch at each node would wait for each)
    double v[L], w[kResHalo], v2[L], w2[kResHalo];
    cells([&](auto z) FEM_INLINE { v[z] = v2[z] = 0.0; });
    rows([&](auto z, uint32_t i) FEM_INLINE { v[z] = dld(T1, i); });
    halo([&](auto k, int) FEM_INLINE { w[k] = dld(T1, B.hnode[k]); });
    if (!S.guess_prev) {
      rows([&](auto z, uint32_t i) FEM_INLINE { v2[z] = dld(T2, i); });
      halo([&](auto k, int) FEM_INLINE { w2[k] = dld(T2, B.hnode[k]); });
    }
    if (zero) {
      rows([&](auto z, uint32_t i) FEM_INLINE { v[z] = (gld(S.pinv64, i) == 0.0) ? v[z] : 0.0; });
      halo([&](auto k, int) FEM_INLINE { w[k] = (gld(S.pinv64, B.hnode[k]) == 0.0) ? w[k] : 0.0; });
    } else if (!S.guess_prev) {
      cells([&](auto z) FEM_INLINE { v[z] = fma(2.0, v[z], -v2[z]); });
      halo([&](auto k, int) FEM_INLINE { w[k] = fma(2.0, w[k], -w2[k]); });
    }
    halo([&](auto k, int) FEM_INLINE { w[k] = ((B.hmask >> k) & 1u) ? w[k] : 0.0; });
    __builtin_amdgcn_sched_barrier(0);
    cells([&](auto z) FEM_INLINE {
      const double t = B.ok ? v[z] : 0.0;
      if constexpr (kMixed)
        x64[z] = t;
      else
        x[z] = t;
      own64[z] = t;
    });
    halo([&](auto k, int o) FEM_INLINE { D64[o] = w[k]; });
    if constexpr (!CHEB)
      fill_coefficients<double, L, false>(B, g, S.s, x0, y0, z0, S.rhoc64, S.k64, S.sa64, S.sbA64, C64);
    its = sweeps = 0;
    ph = kResidual;
  };
  // A vector of the chain: to its exchange, to the column and its halo
  // (is_free: the block has read the vector before it).
  auto chain_vector = [&](int k, bool is_free, const V (&v)[L]) FEM_INLINE {
    U* const E = reinterpret_cast<U*>(S.EC[k]);
    put(E, [&](auto z) FEM_INLINE { return v[z]; });
    if (!is_free) __syncthreads();
    V* const own = column(D + chain_at);
    cells([&](auto z) FEM_INLINE { own[z] = v[z]; });
    V h[kResHalo];
    halo([&](auto k, int) FEM_INLINE { h[k] = V(0); });
    meet_halo<V>(M, E, B, h, &lost);
    halo([&](auto k, int o) FEM_INLINE { D[chain_at + o] = h[k]; });
  };
  // d_0 = P^-1 r / c of the chain that preconditions r.
  auto start_chain = [&]() FEM_INLINE {
    if constexpr (CHEB) {
      cells([&](auto z) FEM_INLINE {
        cr[z] = r[z];
        y[z] = (p[z] * r[z]) * S.ch_inv_c;
      });
      chain_vector(0, true, y);
      ck = 1;
      chain_of = ph;
      ph = kChain;
    }
  };
  // Behind a sum that ends a chain: every block has read the chain's exchanges.
  auto clear_chain = [&]() FEM_INLINE {
    for (int k = 0; k < S.chain; ++k) clear_surface<V, L>(B, reinterpret_cast<U*>(S.EC[k]));
  };
  // How an iteration goes on (kLost: the launch ends).
  enum { kLost, kReplacing, kStepped, kGoOn, kDone };
  auto prec = [&](auto z) FEM_INLINE -> V {  // P^-1 r
    if constexpr (CHEB)
      return y[z];
    else
      return p[z] * r[z];
  };
  // q = A d is known: alpha, then x and r, or the first half of a replacement.
  auto step_along = [&]() FEM_INLINE -> int {
    V* const own = column(D);
    double part = 0.0;
    cells([&](auto z) FEM_INLINE { part += (double)own[z] * (double)q[z]; });
    const double dq = plain_sum(part);
    if (uniform(lost)) return kLost;
    if (timed) clk.summed(lead, S.out);
    const double a = delta / dq;
    if (!(dq > 0.0) || !isfinite(dq) || !isfinite(a)) {
      status = kStatusBreakdown;
      return kLost;
    }
    alpha = uniform((V)a);
    const bool rep = R > 0 && j % R == 0;
    ++j;
    if (rep) {  // x += alpha d, r = b - A x: x takes d's place in D, d waits in r and (its halo) in memory
      if (timed) clk.replacement(lead, S.out);
      cells([&](auto z) FEM_INLINE { r[z] = own[z]; });
      cells([&](auto z) FEM_INLINE {
        x[z] = fma(alpha, r[z], x[z]);
        own[z] = x[z];
      });
      put(EX, [&](auto z) FEM_INLINE { return x[z]; });
      V hx[kResHalo];
      halo([&](auto k, int o) FEM_INLINE { hx[k] = V(0); });
      meet_halo<V>(M, EX, B, hx, &lost);
      V* const stash = static_cast<V*>(S.stash);
      const uint32_t stash_at = blk * M.nt + here((uint32_t)threadIdx.x);
      halo([&](auto k, int o) FEM_INLINE { gst(stash, stash_at + k * M.G * M.nt, D[o]); });
      halo([&](auto k, int o) FEM_INLINE { D[o] = hx[k]; });
      ph = kReplace;
      return kReplacing;
    }
    cells([&](auto z) FEM_INLINE {
      const V rr = fma(-alpha, q[z], r[z]);
      r[z] = (here(p[z]) == V(0)) ? V(0) : rr;
      x[z] = fma(alpha, own[z], x[z]);
    });
    return kStepped;
  };
  // r is new: delta = r^T P^-1 r with P^-1 r of the halo, the stop test, the
  // next direction (first: of a solve; replaced: r has been replaced).
  auto turn = [&](bool first, bool replaced) FEM_INLINE -> int {
    put(E0, [&](auto z) FEM_INLINE { return prec(z); });
    double part = 0.0;
    cells([&](auto z) FEM_INLINE { part += (double)r[z] * (double)prec(z); });
    const double now = meet_sum<false, V, true>(M, mlds, part, E0, B, hv, &lost, []() {});
    if (uniform(lost)) return kLost;
    {
      U* t = E0;
      E0 = E1;
      E1 = E2;
      E2 = t;
      fresh = true;
    }
    if constexpr (CHEB) clear_chain();
    if (timed && !first) clk.updated(lead, S.out, replaced);
    if (replaced) clear_surface<V, L>(B, EX);
    bool done;
    if (first) {
      tol = uniform((kMixed || stop_rule == 1) ? rt2 * now : rt2 * delta_b);
      done = max_iter <= 0 || !(now > tol);
    } else {
      beta = uniform((V)(now / delta));
      done = !(now > tol) || j >= max_iter;
    }
    delta = now;
    if (!isfinite(now)) {
      status = kStatusBreakdown;
      return kLost;
    }
    if (!done) {
      V* const own = column(D);
      // d = P^-1 r + beta d on the brick and its halo (the first d is P^-1 r)
      if (first) {
        cells([&](auto z) FEM_INLINE { own[z] = prec(z); });
        halo([&](auto k, int o) FEM_INLINE { D[o] = hv[k]; });
      } else {  // (all reads before the first write, which could be of the same place for all the compiler knows)
        V v[L], w[kResHalo];
        cells([&](auto z) FEM_INLINE { v[z] = own[z]; });
        halo([&](auto k, int o) FEM_INLINE { w[k] = D[o]; });
        cells([&](auto z) FEM_INLINE { own[z] = fma(beta, v[z], prec(z)); });
        halo([&](auto k, int o) FEM_INLINE { D[o] = fma(beta, w[k], hv[k]); });
      }
      return kGoOn;
    }
    return kDone;
  };
  start_step();
  for (;;) {
    __syncthreads();
    double acc[L];
    if (kMixed && ph <= kResidual) {
      apply(D64, C64, acc);
    } else {
      if (CHEB && timed && ph == kDirection) clk.direction(lead, S.out);
      apply(D + (CHEB && ph == kChain ? chain_at : 0), C, q);
    }
    auto result = [&](auto z) FEM_INLINE -> double {
      if constexpr (kMixed)
        return acc[z];
      else
        return q[z];
    };

    if (ph == kRhs) {  // b = L T^{n-1} + dt s F, delta_b
      const double fs = S.fs[m];
      double part = 0.0;
      double bb[L];
      rows([&](auto z, uint32_t i) FEM_INLINE { bb[z] = gld(S.F, i); });
      rows([&](auto z, uint32_t i) FEM_INLINE {
        bb[z] = fma(fs, bb[z], result(z));
        if (B.ok) gst(S.b, i, bb[z]);
      });
      if (S.lift) rows([&](auto z, uint32_t i) FEM_INLINE { bb[z] = bb[z] - gld(S.lift, i); });
      rows([&](auto z, uint32_t i) FEM_INLINE {
        if constexpr (CHEB) {
          r[z] = B.ok ? bb[z] : 0.0;
        } else {
          const double t = bb[z] * (gld(S.pinv64, i) * bb[z]);
          part += B.ok ? t : 0.0;
        }
      });
      if constexpr (CHEB) {  // delta_b in the preconditioner's norm: r holds b - lift for the chain
        __syncthreads();  // L's coefficients have been read
        fill_coefficients<double, L, false>(B, g, S.s, x0, y0, z0, S.rhoc64, S.k64, S.sa64, S.sbA64, C64);
        start_chain();
        continue;
      }
      delta_b = plain_sum(part);
      if (uniform(lost)) break;
      start_solve();
      continue;
    }

    bool finished = false;  // the step's solve has ended
    bool chained = false;   // the chain has preconditioned r
    if (CHEB && ph == kChain) {  // step ck of the chain (EpiCheb's arithmetic)
      if constexpr (CHEB) {
        const double a = S.ch_a[ck - 1], b = S.ch_b[ck - 1];
        V* const own = column(D + chain_at);
        V d[L];
        cells([&](auto z) FEM_INLINE {
          cr[z] = cr[z] - q[z];
          d[z] = fma(a, own[z], b * (p[z] * cr[z]));
          y[z] = y[z] + d[z];
        });
        if (ck < S.chain) {
          chain_vector(ck, false, d);
          ++ck;
          continue;
        }
        ph = chain_of;
        if (ph == kRhs) {
          double part = 0.0;
          cells([&](auto z) FEM_INLINE { part += r[z] * y[z]; });
          delta_b = plain_sum(part);
          if (uniform(lost)) break;
          clear_chain();
          start_solve();
          (void)plain_sum(0.0);  // (the chain is used again before the next sum)
          if (uniform(lost)) break;
          continue;
        }
        chained = true;
      }
    } else if (ph == kResidual) {  // r = b - A x of the initial guess, or after a correction (mixed form)
      if constexpr (!kMixed) {
        double bv[L];  // (r is written as a whole: it is not live before)
        cells([&](auto z) FEM_INLINE { bv[z] = 0.0; });
        rows([&](auto z, uint32_t i) FEM_INLINE { bv[z] = gld(S.b, i); });
        cells([&](auto z) FEM_INLINE { r[z] = (here(p[z]) == 0.0) ? 0.0 : bv[z] - q[z]; });
        rt2 = rtol2;
      } else {
        double part = 0.0, pv[L];
        cells([&](auto z) FEM_INLINE { pv[z] = r64[z] = 0.0; });
        rows([&](auto z, uint32_t i) FEM_INLINE {
          pv[z] = gld(S.pinv64, i);
          r64[z] = gld(S.b, i);
        });
        cells([&](auto z) FEM_INLINE {
          const double pz = B.ok ? pv[z] : 0.0;
          r64[z] = (pz == 0.0) ? 0.0 : r64[z] - acc[z];
          part += r64[z] * (pz * r64[z]);
        });
        odelta = plain_sum(part);
        if (uniform(lost)) break;
        const bool initial = sweeps == 0;
        if (initial) {
          odelta0 = odelta;
          otol = uniform(stop_rule == 1 ? rtol2 * odelta : rtol2 * delta_b);
        } else {
          clear_surface<double, L>(B, reinterpret_cast<U64*>(S.EX64));
            }
        if (!isfinite(odelta)) {
          status = kStatusBreakdown;
          break;
        }
        finished = (initial && max_iter <= 0) || !(odelta > otol) || sweeps >= S.max_refine;
        if (!finished) {  // inner solve of A e = r64 to half the reduction the FP64 rule still needs
          const double ref = stop_rule == 1 ? odelta0 : delta_b;
          const double need = odelta > 0.0 ? 0.5 * sqrt(rtol2 * ref / odelta) : 1.0;
          const double irt = fmin(0.5, fmax(S.inner_rtol, need));
          rt2 = uniform(irt * irt);
          fill_coefficients<float, L, true>(B, g, S.s, x0, y0, z0, S.rhoc32, S.k32, S.sa32, S.sbA32, C);
          cells([&](auto z) FEM_INLINE {
            r[z] = (float)r64[z];
            x[z] = 0.0f;
          });
        }
      }
      first = true;
      j = 0;
    } else if (CHEB && ph == kDirection) {
      const int next = step_along();
      if (next == kLost) break;
      if (next == kReplacing) continue;
    } else {  // kReplace
      __syncthreads();  // x has been read
      V* const own = column(D);
      cells([&](auto z) FEM_INLINE { own[z] = r[z]; });
      V rhs[L];
      cells([&](auto z) FEM_INLINE {
        if constexpr (kMixed)
          rhs[z] = (float)r64[z];
        else
          rhs[z] = V(0);
      });
      if constexpr (!kMixed) rows([&](auto z, uint32_t i) FEM_INLINE { rhs[z] = gld(S.b, i); });
      cells([&](auto z) FEM_INLINE { r[z] = (here(p[z]) == V(0)) ? V(0) : rhs[z] - q[z]; });
      const V* const stash = static_cast<const V*>(S.stash);
      const uint32_t stash_at = blk * M.nt + here((uint32_t)threadIdx.x);
      halo([&](auto k, int o) FEM_INLINE {
        D[o] = gld(stash, stash_at + k * M.G * M.nt);
      });
    }

    if (CHEB && !chained) {
      start_chain();
      continue;
    }
    if (!finished) {
      int next = turn(first, ph == kReplace);
      first = false;
      // The iterations, in a loop of their own with its own copy of the march:
      // joined with the other phases, every one moved the brick's registers
      // and spilled scalars to where the phases meet (17^3 6.84 -> 6.55 us per
      // iteration, 49^3 6.95 -> 6.71, 201 x 201 x 26 mixed 10.8 -> 10.2).
      // The chain's form, whose registers are fuller, keeps one march.
      if constexpr (!CHEB)
        while (next == kGoOn) {
          __syncthreads();
          if (timed) clk.direction(lead, S.out);
          apply(D, C, q);
          next = step_along();
          if (next == kStepped) next = turn(false, false);
        }
      if (next == kLost) break;
      if (next == kGoOn) ph = kDirection;
      if (next != kDone) continue;
      its += j;
      if constexpr (!kMixed) {
        odelta = delta;
        otol = tol;
      } else {  // x64 += e on the brick and, through the exchange, on its halo; then its residual
        __syncthreads();
        double* const own64 = column(D64);
        cells([&](auto z) FEM_INLINE {
          x64[z] = fma(1.0, (double)x[z], x64[z]);
          own64[z] = x64[z];
        });
        U64* const EX64 = reinterpret_cast<U64*>(S.EX64);
        put(EX64, [&](auto z) FEM_INLINE { return x64[z]; });
        fill_coefficients<double, L, true>(B, g, S.s, x0, y0, z0, S.rhoc64, S.k64, S.sa64, S.sbA64, C64);
        halo([&](auto k, int o) FEM_INLINE { hd[k] = 0.0; });
        meet_halo<double>(M, EX64, B, hd, &lost);
        halo([&](auto k, int o) FEM_INLINE { D64[o] = hd[k]; });
        ++sweeps;
        ph = kResidual;
        continue;
      }
    }

    // ---- end of the step: the new field to memory, its record, the sensors
    if (B.ok)
      rows([&](auto z, uint32_t i) FEM_INLINE {
        double v;
        if constexpr (kMixed)
          v = x64[z];
        else
          v = x[z];
        U64 u;
        __builtin_memcpy(&u, &v, 8);
        dev_st(reinterpret_cast<U64*>(T3), i, u);
      });
    if (lead) S.rec[m] = ResStep{its, sweeps, odelta, delta_b, otol};
    {
      double* t = T3;
      T3 = T2;
      T2 = T1;
      T1 = t;
    }
    ++m;
    bool over = false;
    if (m < S.nsteps || S.nsens > 0) {
      over = plain_sum(lead && wall_clock64() > until ? 1.0 : 0.0) != 0.0;
      if (uniform(lost)) {
        --m;
        break;
      }
    }
    if (S.nsens > 0) {
      const int first_q = (int)blk * M.nt + (int)threadIdx.x, stride = (int)M.G * M.nt;
      for (int s = first_q; s < S.nsens; s += stride)
        S.traces[(size_t)(m - 1) * S.nsens + s] = sensor_value(g, S.xyz, s, [&](uint32_t i) FEM_INLINE { return dld(T1, i); });
    }
    if (m >= S.nsteps || over) break;
    ph = kRhs;
    start_step();
  }
  if (lost && threadIdx.x == 0) dev_st(S.ctl, 1, 1ull);  // the others give up too
  if (lead) {
    (void)dev_add(S.launch, 0, ~0ull);
    ResOut& w = *S.out;
    w.state = lost ? RES_LOST : RES_RAN;
    w.steps = m;
    w.status = status;
  }
}

}  // namespace femheat
