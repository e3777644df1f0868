// Host side of the resident form: see resident_host.hpp.
#include "resident_host.hpp"

#include <algorithm>
#include <array>
#include <condition_variable>
#include <mutex>


namespace femheat {

const void* resident_kernel_f64(int kind, int planes);    // resident_f64.hip
const void* resident_kernel_mixed(int kind, int planes);  // resident_mixed.hip
const void* resident_kernel_cheb(int kind, int planes);   // resident_cheb.hip

namespace {

// Planes of a brick the kernels are built for: odd, so that the columns of a
// wave lie in distinct LDS banks (see kResPitch).
constexpr int kResPlanes[] = {3, 5, 9};

constexpr int kMaxDevices = 64;

struct GateState {
  std::mutex mu;
  std::condition_variable cv;
  int taken = 0, total = 0;
  uint64_t next = 0, serving = 0;
};
std::array<GateState, kMaxDevices>& gates() {
  static std::array<GateState, kMaxDevices> g;
  return g;
}

}  // namespace

// Estimated microseconds of an iteration of a cut, a linear fit to 250 cuts
// measured on grids of 17^3, 49^3, 58 x 84 x 40 (stretched), 91 x 91 x 31
// (tetrahedra) and 101^3 nodes (MI355X, FP64): the two sums take 3.8 us and
// 6.7 ns per block, a layer of the march 0.38 us with one wave per SIMD and
// 0.55 us with two, a halo node that a brick shares across an x-face 4.5 ns
// (its values lie a row apart) and any other 0.7 ns.  So full rows and low
// bricks win where they fit: 49^3 as 49 x 5 x 3 took 6.9 us, as 25 x 10 x 5
// 7.8 us, as 49 x 10 x 9 10.3 us; 17^3 as 17 x 6 x 3 6.7 us, in two bricks
// 11.6 us.  (These figures are the fit's, which ranks the cuts.  Iterations and
// waits have become 4 to 15% shorter since, on every cut: the chosen ones take
// 5.9 us on 49^3 and 5.8 us on 17^3 now.)  A simulation alone takes the cut with the shortest iteration; a
// batch member the one with the least iteration time per compute unit, as
// other members fill the rest.  A step of the Chebyshev preconditioner's chain
// is another march and an exchange without a sum (1.9 us): at degree 3 the
// resident form takes 18.0 us per iteration on 65^3 nodes (two-kernel form 45),
// 12.5 us on 21^3 (38.6), 27.4 us on 87 x 87 x 85 (55.8), and every cut that
// fits is faster than the two-kernel form.
ResShape resident_shape(const Geom& g, const fem_opts& o, bool batched, int cus) {
  ResShape best{};
  double best_t = 0.0;
  // the form is Algorithm 1 with two sums per iteration, the chain of the
  // Chebyshev preconditioner as long as its exchange vectors; a caller that names a gather tile, or another form of the
  // iteration, gets the kernels it names
  const bool cheb = o.precond == FEM_PRECOND_CHEBYSHEV;
  if ((cheb && o.cheb_degree - 1 > kResChain) || (o.flags & (FEM_ONE_REDUCTION | FEM_ONE_KERNEL)) || o.tile_x != 0 ||
      o.tile_y != 0 || o.tile_z != 0)
    return best;
  const int limit = std::min(cus, kResBlocks);
  for (int nbx = 1; nbx <= g.px; ++nbx) {
    const int a = (g.px + nbx - 1) / nbx;
    if ((g.px + a - 1) / a != nbx || a > kResThreads) continue;
    if (nbx > limit) break;
    for (int nby = 1; nby <= g.py; ++nby) {
      const int b = (g.py + nby - 1) / nby;
      if (nbx * nby > limit) break;
      if ((g.py + b - 1) / b != nby || a * b > kResThreads) continue;
      const int nt = (a * b + 63) / 64 * 64;
      for (int c : kResPlanes) {
        const int nbz = (g.pz + c - 1) / c;
        const int64_t nblk = (int64_t)nbx * nby * nbz;
        if (nblk > limit || res_lds(a, b, c, cheb ? RES_CHEB : RES_F64) > kResLds) continue;
        const int halo = 2 * (a + 2) * (b + 2) + c * (2 * (a + 2) + 2 * b);
        const int per = (halo + nt - 1) / nt;
        if (per > kResHalo) continue;
        const int xface = nbx > 1 ? 2 * b * c : 0, rest = 2 * (a + 2) * (b + 2) + 2 * (a + 2) * c;
        const double march = (c + 1) * (nt <= 256 ? 0.38 : 0.55), halo_us = 0.0045 * xface + 0.0007 * rest;
        double iter = (nblk > 1 ? 3.8 + 0.0067 * (double)nblk + halo_us : 1.0) + march;
        if (cheb) iter += (o.cheb_degree - 1) * ((nblk > 1 ? 1.9 + halo_us : 0.5) + march);
        const double t = batched ? iter * (double)nblk : iter;
        if (best.nblk == 0 || t < best_t) {
          best = ResShape{a, b, c, nbx, nby, nbz, (uint32_t)nblk, nt};
          best_t = t;
        }
      }
    }
  }
  return best;
}

bool resident_member(const fem_grid& grid, const fem_opts& o, bool batched, int cus) {
  Geom g{};
  g.px = grid.nx + 1;
  g.py = grid.ny + 1;
  g.pz = grid.nz + 1;
  return resident_shape(g, o, batched, cus).nblk > 0;
}

hipError_t resident_launch(ResForm form, int kind, int planes, uint32_t blocks, int nthreads, size_t lds,
                           hipStream_t stream, const ResSim* sims, const uint2* table) {
  const void* fn = form == RES_MIXED  ? resident_kernel_mixed(kind, planes)
                   : form == RES_CHEB ? resident_kernel_cheb(kind, planes)
                                      : resident_kernel_f64(kind, planes);
  if (!fn) return hipErrorInvalidValue;
  // the same limit in every call: it is the kernel's, and another thread may be
  // about to launch the kernel with more LDS than this launch takes
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kResLds);
  if (e != hipSuccess) return e;
  void* args[] = {&sims, &table};
  return hipLaunchKernel(fn, dim3(blocks), dim3((uint32_t)nthreads), args, lds, stream);
}

// Blocks over the nodes of a simulation (x), and simulations (y): the kernel
// takes those past the grid in further rounds, as a batch may hold more than a
// grid has rows (65535).
dim3 resident_reset_grid(uint32_t n, uint32_t max_nodes) {
  const uint32_t y = std::min<uint32_t>(std::max<uint32_t>(n, 1), 1024);
  const uint32_t x = std::min<uint32_t>((max_nodes + 255) / 256, std::max<uint32_t>(8, 2048 / y));
  return dim3(std::max<uint32_t>(1, x), y);
}

ResidentGate::ResidentGate(int device, int cus, int want) : device_(device), want_(std::min(want, cus)) {
  GateState& s = gates()[(size_t)device];
  std::unique_lock<std::mutex> lk(s.mu);
  s.total = cus;
  const uint64_t me = s.next++;
  s.cv.wait(lk, [&] { return s.serving == me && s.taken + want_ <= s.total; });
  s.taken += want_;
  ++s.serving;
  s.cv.notify_all();
}

ResidentGate::~ResidentGate() {
  GateState& s = gates()[(size_t)device_];
  {
    std::lock_guard<std::mutex> lk(s.mu);
    s.taken -= want_;
  }
  s.cv.notify_all();
}

}  // namespace femheat
