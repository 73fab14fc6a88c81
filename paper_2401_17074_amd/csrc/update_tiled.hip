// Dispatch of the tiled update over the storage formats, and its work list.
#include "tslb_tiles.h"

namespace tslb {

using namespace tile;

hipError_t tiled_schedule(const Geometry& g, std::vector<int4>& seg, int& grid, int& nseg, long long& steps) {
    const int columns = ((g.n[0] + TX - 1) / TX) * ((g.n[1] + TY - 1) / TY);
    const int resident = (compute_units() * kBlocksPerCu + 7) & ~7;
    Schedule s = build_schedule(columns, g.n[2], resident);
    if (s.grid < 8 || s.nseg < 1) return hipErrorInvalidValue;
    seg = std::move(s.seg);
    grid = s.grid;
    nseg = s.nseg;
    steps = s.cost;
    return hipSuccess;
}

hipError_t launch_update_tiled_f32(const void* in, void* out, const StepParams& p, hipStream_t s);
hipError_t launch_update_tiled_f16(const void* in, void* out, const StepParams& p, hipStream_t s);
hipError_t launch_update_tiled_bf16(const void* in, void* out, const StepParams& p, hipStream_t s);
bool tiled_writes_x_ghosts_f32(const StepParams& p);
bool tiled_writes_x_ghosts_f16(const StepParams& p);
bool tiled_writes_x_ghosts_bf16(const StepParams& p);

bool tiled_writes_x_ghosts(int storage, const StepParams& p) {
    switch (storage) {
    case 0: return tiled_writes_x_ghosts_f32(p);
    case 1: return tiled_writes_x_ghosts_f16(p);
    case 2: return tiled_writes_x_ghosts_bf16(p);
    }
    return false;
}

hipError_t launch_update_tiled(int storage, const void* in, void* out, const StepParams& p, hipStream_t s) {
    switch (storage) {
    case 0: return launch_update_tiled_f32(in, out, p, s);
    case 1: return launch_update_tiled_f16(in, out, p, s);
    case 2: return launch_update_tiled_bf16(in, out, p, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace tslb
