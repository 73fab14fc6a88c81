// Tiled adjoint with tiles of 12 rows, and its dispatch over the tiles of the
// handle's work list (see tiled_schedule).
#include "adjoint_tiled_kernel.h"

namespace tslb {
hipError_t launch_adjoint_tiled_rows8(const float* st0, const float* st1, const float* lam1, float* lam0, float* dg,
                                      const StepParams& p, hipStream_t s);

hipError_t launch_adjoint_tiled(const float* st0, const float* st1, const float* lam1, float* lam0, float* dg,
                                const StepParams& p, hipStream_t s) {
    return p.sched_other_rows ? launch_adjoint_tiled_rows8(st0, st1, lam1, lam0, dg, p, s)
                         : launch_adjoint(st0, st1, lam1, lam0, dg, p, s);
}
}  // namespace tslb
