// Dispatch of the tiled update over the storage formats, and its work list.
#include "tslb_tiles.h"

namespace tslb {

using namespace tile;

hipError_t launch_update_tiled_f32(const void* in, void* out, const StepParams& p, hipStream_t s);
hipError_t launch_update_tiled_f16(const void* in, void* out, const StepParams& p, hipStream_t s);
hipError_t launch_update_tiled_bf16(const void* in, void* out, const StepParams& p, hipStream_t s);
bool tiled_writes_x_ghosts_f32(const StepParams& p);
bool tiled_writes_x_ghosts_f16(const StepParams& p);
bool tiled_writes_x_ghosts_bf16(const StepParams& p);

int tiled_columns_f32(const Geometry& g);
int tiled_columns_f16(const Geometry& g);
int tiled_columns_bf16(const Geometry& g);

hipError_t tiled_schedule(int storage, const Geometry& g, std::vector<int4>& seg, int& grid, int& nseg,
                          long long& steps) {
    const int columns = storage == 0 ? tiled_columns_f32(g) : storage == 1 ? tiled_columns_f16(g) : tiled_columns_bf16(g);
    const int resident = (compute_units() + 7) & ~7;  // one block per CU
    Schedule s = build_schedule(columns, g.n[2], resident);
    if (s.grid < 8 || s.nseg < 1) return hipErrorInvalidValue;
    seg = std::move(s.seg);
    grid = s.grid;
    nseg = s.nseg;
    steps = s.cost;
    return hipSuccess;
}

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
