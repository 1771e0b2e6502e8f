// Spread sampler instances: proposal mode PM_BF16X1.
#include "sampler_spread.hpp"

namespace dmala {
hipError_t launch_spread_bf16x1(const Shape& sh, const SamplerArgs& a, hipStream_t s, const Persist* p, int gn, KernelCfg* cfg) {
  return launch_spread_pm<PM_BF16X1>(sh, a, s, p, gn, cfg);
}
}  // namespace dmala
