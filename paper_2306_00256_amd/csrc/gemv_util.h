// Loss derivative shared by the minibatch-gradient kernels.
#pragma once
#include <hip/hip_runtime.h>

#include "ceca.h"

namespace ceca {

// Loss derivative at margin m with target / label t, already divided by the batch size.
__device__ __forceinline__ float loss_coef(int kind, float m, float t, float scale) {
  // LOGISTIC: -t * sigma(-t m) with sigma(-u) = 1 / (1 + e^u); e^u = inf gives 0, e^u = 0 gives 1
  const float cf = (kind == CECA_LOSS_LSQ) ? (m - t) : (-t / (1.0f + expf(t * m)));
  return cf * scale;
}

}  // namespace ceca
