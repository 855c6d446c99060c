// kernels_adex_exp_plastic.hip -- step kernels of networks with AdEx neurons (exponential ports only, plastic synapses).
#include "step_dev.h"

namespace snn {

void launch_adex_exp_plastic(const NetDev& nd, dim3 grid, hipStream_t s, hipEvent_t start, hipEvent_t stop, uint32_t rel,
                    bool lif) {
  launch_adex<1, true>(nd, grid, s, start, stop, rel, lif);
}

}  // namespace snn
