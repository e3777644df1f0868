// Host side of the resident form (resident.hpp): the cut of a grid into
// bricks, the launches, and the gate that keeps the process's resident
// kernels from asking for more compute units than the device has.
#pragma once

#include "resident_types.hpp"

namespace femheat {

// The cut for a simulation (nblk = 0: it takes the two-kernel form).  Depends
// on the grid, the options, the launch kind and the device alone.
ResShape resident_shape(const Geom& g, const fem_opts& o, bool batched, int cus);

// One launch over `blocks` bricks of simulations with the same element kind
// and the same planes per brick.
hipError_t resident_launch(ResForm form, int kind, int planes, uint32_t blocks, int nthreads, size_t lds,
                           hipStream_t stream, const ResSim* sims, const uint2* table);
// Prepares the launches of a pass: n simulations of at most max_nodes nodes.
hipError_t resident_reset(hipStream_t stream, const ResSim* sims, uint32_t n, ResForm form, uint32_t max_nodes);
dim3 resident_reset_grid(uint32_t n, uint32_t max_nodes);

// Compute units of one device, taken by resident launches of this process:
// two kernels whose blocks wait for blocks of their own must both fit, or
// each could hold what the other waits for.  In arrival order.
class ResidentGate {
 public:
  ResidentGate(int device, int cus, int want);
  ~ResidentGate();
  ResidentGate(const ResidentGate&) = delete;
  ResidentGate& operator=(const ResidentGate&) = delete;

 private:
  int device_, want_;
};

}  // namespace femheat
