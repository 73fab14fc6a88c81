// FP16-storage instantiations of the tiled update with tiles of 13 rows (see
// tiled_schedule).
#undef TSLB_TILE_Y
#define TSLB_TILE_Y 13
#include "update_tiled_kernel.h"

namespace tslb {
hipError_t launch_update_tiled_rows13_f16(const void* in, void* out, const StepParams& p, hipStream_t s) {
    return launch_s<StoreF16>(in, out, p, s);
}
int tiled_columns_rows13_f16(const Geometry& g) { return tile_columns(g); }
}  // namespace tslb
