// Tiled adjoint with tiles of 8 rows (see tiled_schedule).
#undef TSLB_TILE_Y
#define TSLB_TILE_Y 8
#include "adjoint_tiled_kernel.h"

namespace tslb {
hipError_t launch_adjoint_tiled_rows8(const float* st0, const float* st1, const float* lam1, float* lam0, float* dg,
                                      const StepParams& p, hipStream_t s) {
    return launch_adjoint(st0, st1, lam1, lam0, dg, p, s);
}
}  // namespace tslb
