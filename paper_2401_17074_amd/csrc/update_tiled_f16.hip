// FP16-storage instantiations of the tiled update.
#include "update_tiled_kernel.h"

namespace tslb {
hipError_t launch_update_tiled_f16(const void* in, void* out, const StepParams& p, hipStream_t s) {
    return launch_s<StoreF16>(in, out, p, s);
}
int tiled_columns_f16(const Geometry& g) { return tile_columns(g); }
bool tiled_writes_x_ghosts_f16(const StepParams& p) { return writes_x_ghosts<StoreF16>(p); }
}  // namespace tslb
