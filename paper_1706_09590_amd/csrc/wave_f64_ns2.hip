// Instantiations of the wave variant of the fused RK stage for double state, 2 electronic states.
#include "stage_wave.hpp"

namespace qhfpe {
hipError_t launch_stage_wave_f64_ns2(int np, const StageArgs& a, int nblocks, hipStream_t s) {
  return launch_stage_wave<double, 2>(np, a, nblocks, s);
}
}  // namespace qhfpe
