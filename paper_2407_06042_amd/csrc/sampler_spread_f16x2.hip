// Spread sampler instances: proposal mode PM_F16X2.
#include "sampler_spread.hpp"

namespace dmala {
hipError_t launch_spread_f16x2(const Shape& sh, const SamplerArgs& a, hipStream_t s, const Persist* p, int gn, KernelCfg* cfg) {
  return launch_spread_pm<PM_F16X2>(sh, a, s, p, gn, cfg);
}
}  // namespace dmala
