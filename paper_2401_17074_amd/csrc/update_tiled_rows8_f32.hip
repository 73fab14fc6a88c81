// FP32-storage instantiations of the tiled update with tiles of 8 rows (see
// tiled_schedule).
#undef TSLB_TILE_Y
#define TSLB_TILE_Y 8
#include "update_tiled_kernel.h"

namespace tslb {
hipError_t launch_update_tiled_rows8_f32(const void* in, void* out, const StepParams& p, hipStream_t s) {
    return launch_s<StoreF32>(in, out, p, s);
}
int tiled_columns_rows8_f32(const Geometry& g) { return tile_columns(g); }
}  // namespace tslb
