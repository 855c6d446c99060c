// kernels_adex_beta.hip -- step kernels of networks with AdEx neurons (beta ports).
#include "step_dev.h"

namespace snn {

void launch_adex_beta(const NetDev& nd, dim3 grid, hipStream_t s, hipEvent_t start, hipEvent_t stop, uint32_t rel,
                    bool lif) {
  launch_adex<2, false>(nd, grid, s, start, stop, rel, lif);
}

}  // namespace snn
