// Scalars of a step that a stage update advances (one thread of its kernel).
#pragma once

#include "kernels.h"

namespace wb {

// Bound on the move of every particle by the stage update just made (Sec.
// 2.3), added to sc->disp.  Stage 1: x1 - x0 = dt (U0 + dU0), |U0| <= U_max0
// and the shifting velocity is clamped to U_max0 / 2, so |x1 - x0| <= 1.5 dt
// U_max0.  Stage 2: x2 - x1 = (dt (U1 + dU1) - dt (U0 + dU0)) / 2, so
// |x2 - x1| <= 0.75 dt (U_max0 + U_max1).  The relative margin covers the
// rounding of the bound and of FP32 velocities.
__device__ __forceinline__ void disp_add(Scalars *sc, int stage) {
  const double dt = sc->dt;
  if (stage == 1) {
    sc->umax1 = sc->umax;
    sc->disp += 1.5 * dt * sc->umax * (1.0 + 1e-6);
  } else {
    sc->disp += 0.75 * dt * (sc->umax1 + sc->umax) * (1.0 + 1e-6);
  }
}

// The step's scalars after a stage update, by one thread of its kernel (which
// reads none of them but dt) or by a launch of its own.
__device__ void finish_stage(Scalars *sc, int stage, int finish) {
  if (finish & kFinishDisp) disp_add(sc, stage);
  if (finish & kFinishStep) {
    sc->t = sc->t + sc->dt;
    sc->steps += 1.0;
  }
}

}  // namespace wb
