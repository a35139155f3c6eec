// The proximal step, shared by the SGD step loops.
#pragma once
#include "../../include/zipml.h"
#include "zipml_device.h"

namespace zipml {

// Proximal operator of lr * R at v, coordinate-wise (Sec. 2, x <- prox_{gamma R}(x - gamma g)):
// l1 norm -> soft threshold at lr * coef; coef/2 ||x||^2 -> v / (1 + lr * coef); the constraint
// ||x||_inf <= coef -> clamp.  None of them increases |v|, so the magnitude bounds that the step
// loops track for the model stay valid.
__device__ __forceinline__ float apply_prox(float v, int kind, float lr, float coef)
{
    if (kind == ZIPML_PROX_L1) {
        const float t = lr * coef;
        return v > t ? v - t : v < -t ? v + t : 0.0f;
    }
    if (kind == ZIPML_PROX_L2SQ) return __fdiv_rn(v, 1.0f + lr * coef);
    if (kind == ZIPML_PROX_BOX) return fminf(fmaxf(v, -coef), coef);
    return v;
}

}  // namespace zipml
