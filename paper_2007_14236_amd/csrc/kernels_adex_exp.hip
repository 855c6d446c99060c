// kernels_adex_exp.hip -- step kernels of networks with AdEx neurons (exponential ports only).
#include "step_dev.h"

namespace snn {

void launch_adex_exp(const NetDev& nd, dim3 grid, hipStream_t s, hipEvent_t start, hipEvent_t stop, uint32_t rel,
                    bool lif) {
  launch_adex<1, false>(nd, grid, s, start, stop, rel, lif);
}

}  // namespace snn
