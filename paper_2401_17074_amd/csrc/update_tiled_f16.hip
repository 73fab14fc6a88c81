// FP16-storage instantiations of the tiled update.
// Tile of 13 rows: 16 waves a block in place of 15, so fewer halo columns per
// node, which the arithmetic of 16-bit storage feels (us per step, 12 / 13
// rows: 512 x 256 x 256 channel FP16 393 / 383, 384 x 192 x 192 180 / 175,
// 288 x 96 x 192 85 / 77, 192 x 64 x 128 25.9 / 23.6; FP32 is bound by memory
// and keeps 12: 512 x 256 x 256 periodic 538 / 557).
#ifndef TSLB_TILE_Y
#define TSLB_TILE_Y 13
#endif
#include "update_tiled_kernel.h"

namespace tslb {
hipError_t launch_update_tiled_f16(const void* in, void* out, const StepParams& p, hipStream_t s) {
    return launch_s<StoreF16>(in, out, p, s);
}
int tiled_columns_f16(const Geometry& g) { return tile_columns(g); }
bool tiled_writes_x_ghosts_f16(const StepParams& p) { return writes_x_ghosts<StoreF16>(p); }
}  // namespace tslb
