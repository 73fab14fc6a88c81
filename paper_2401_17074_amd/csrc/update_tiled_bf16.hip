// BF16-storage instantiations of the tiled update.
#include "update_tiled_kernel.h"

namespace tslb {
hipError_t launch_update_tiled_bf16(const void* in, void* out, const StepParams& p, hipStream_t s) {
    return launch_s<StoreBF16>(in, out, p, s);
}
int tiled_columns_bf16(const Geometry& g) { return tile_columns(g); }
bool tiled_writes_x_ghosts_bf16(const StepParams& p) { return writes_x_ghosts<StoreBF16>(p); }
}  // namespace tslb
