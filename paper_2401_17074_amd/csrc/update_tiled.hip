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
hipError_t launch_update_tiled_rows8_f32(const void* in, void* out, const StepParams& p, hipStream_t s);
hipError_t launch_update_tiled_rows13_f16(const void* in, void* out, const StepParams& p, hipStream_t s);
hipError_t launch_update_tiled_rows13_bf16(const void* in, void* out, const StepParams& p, hipStream_t s);
int tiled_columns_rows8_f32(const Geometry& g);
int tiled_columns_rows13_f16(const Geometry& g);
int tiled_columns_rows13_bf16(const Geometry& g);

// Tiles of 12 rows, or of another height:
// FP32, 8 rows: a block has 11 waves in place of 15, so each of its plane-steps
// is shorter, and it needs more of them.  Taken where it needs at most one
// more: on small grids, where the chain of steps is the time, and where 8 rows
// divide the grid better (us per step, 12 rows / 8; plane-steps in brackets:
// 64^3 10.1 (4) / 8.7 (4), 64 x 64 x 128 13.6 (6) / 12.2 (6), 80^3 15.3 (7) /
// 17.8 (9), 96^3 18.2 (8) / 20.4 (11); adjoint step of 64^3 11.5 / 10.5).
// 16-bit storage, 13 rows: a block has 16 waves in place of 15, so fewer halo
// columns per node, but no SIMD with a wave less.  Taken where two levels
// exceed the Infinity Cache, with walls always (us per step, 12 rows / 13, FP16:
// channels 512 x 256 x 256 386 / 389, 384 x 192 x 192 179 / 179, 512 x 96 x 400
// 255 / 240, 250^3 216 / 203), without where they save a fifteenth of the
// tile columns (389 x 386 x 86 224 / 205, 96 x 160 x 736 314 / 296; not 512 x 96
// x 400 216 / 228, 160 x 200 x 210 87 / 96, 864 x 120 x 175 237 / 250); or where
// they exceed L2 and 13 rows save 15 % of the plane-steps (200 x 150 x 100 50.4
// / 48.4, jet 160 x 64 x 320 BF16 76.4 / 70.4; not 128^3 30.7 / 33.5).  FP32,
// bound by memory, keeps 12 (512 x 256 x 256 538 / 557).  Levels that fit L2
// keep 12.  The values do not depend on the height (see crosses_up).
hipError_t tiled_schedule(int storage, const Geometry& g, std::vector<int4>& seg, int& grid, int& nseg, int& other_rows,
                          long long& steps) {
    const int resident = (compute_units() + 7) & ~7;  // one block per CU
    const int columns = storage == 0 ? tiled_columns_f32(g) : storage == 1 ? tiled_columns_f16(g) : tiled_columns_bf16(g);
    const int other = storage == 0   ? tiled_columns_rows8_f32(g)
                      : storage == 1 ? tiled_columns_rows13_f16(g)
                                     : tiled_columns_rows13_bf16(g);
    Schedule s;
    other_rows = 0;
    if (storage == 0) {
        s = build_schedule(columns, g.n[2], resident);
        steps = s.cost;
        Schedule s8 = build_schedule(other, g.n[2], resident, s.cost + 1);
        other_rows = s8.grid > 0;
        if (other_rows) s = std::move(s8);
    } else {
        const size_t levels = 2 * 20 * (size_t)g.N;
        const bool walls = (g.lo_solid | g.hi_solid) != 0;
        other_rows = levels > kInfinityCacheBytes && (walls || 15LL * other <= 14LL * columns);
        s = build_schedule(other_rows ? other : columns, g.n[2], resident);
        if (levels > kL2Bytes && levels <= kInfinityCacheBytes) {
            Schedule s13 = build_schedule(other, g.n[2], resident, 17 * s.cost / 20);
            other_rows = s13.grid > 0;
            if (other_rows) s = std::move(s13);
        }
        steps = s.cost;
    }
    if (s.grid < 8 || s.nseg < 1) return hipErrorInvalidValue;
    seg = std::move(s.seg);
    grid = s.grid;
    nseg = s.nseg;
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
    case 0: return p.sched_other_rows ? launch_update_tiled_rows8_f32(in, out, p, s) : launch_update_tiled_f32(in, out, p, s);
    case 1: return p.sched_other_rows ? launch_update_tiled_rows13_f16(in, out, p, s) : launch_update_tiled_f16(in, out, p, s);
    case 2: return p.sched_other_rows ? launch_update_tiled_rows13_bf16(in, out, p, s) : launch_update_tiled_bf16(in, out, p, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace tslb
