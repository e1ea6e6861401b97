// Runs a kernel on the host: see hip/hip_runtime.h.  The waves are scheduled at
// random from a seed.
#pragma once
#include <functional>

namespace emu {

struct Launch {
  unsigned grid = 1, block = 64;
  unsigned long long seed = 1;
  double hold = 0.0;                // chance, per pick, that a wave is then left alone for long
  unsigned held_for = 0;            //   (in picks)
  std::function<unsigned long long(unsigned)> start;   // pick at which a workgroup starts
  int stalled = -1;                 // a workgroup left alone for a while; from then on the
  unsigned long long stall_from = 0, stall_to = 0;     //   clock runs 100,000 times as fast
  unsigned long long limit = 200000000;                // picks; past it the run has failed
  double ticks = 0.02;              // of the wall clock, per pick
};
// kernel(workgroup) is called by every lane.  Returns picks used, 0 past the limit.
unsigned long long run(const Launch& l, const std::function<void(unsigned)>& kernel);

}  // namespace emu
