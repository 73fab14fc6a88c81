// Host-side check of the choice between bricks and tiles (tile::brick_grid):
// prints nx ny nz bricks chosen for the grids given as arguments, on 256
// compute units and FP32 storage.
#include <cstdio>
#include <cstdlib>

#include "tslb_tiles.h"

using namespace tslb;
using namespace tslb::tile;

int main(int argc, char** argv) {
    for (int k = 1; k + 2 < argc; k += 3) {
        Geometry g{};
        for (int d = 0; d < 3; ++d) g.n[d] = atoi(argv[k + d]);
        g.N = (long long)g.n[0] * g.n[1] * g.n[2];
        const int tx = (g.n[0] + TX - 1) / TX;
        const Schedule s = build_schedule(tx * ((g.n[1] + TY - 1) / TY), g.n[2], 256);
        // tiles of 8 rows where they take at most one plane-step more
        const bool rows8 = build_schedule(tx * ((g.n[1] + 7) / 8), g.n[2], 256, s.cost + 1).grid > 0;
        printf("%d %d %d %lld %d %d\n", g.n[0], g.n[1], g.n[2], brick_count(g), (int)brick_grid(0, g, s.cost, rows8, 256),
               (int)brick_grid(1, g, s.cost, rows8, 256));
    }
    return 0;
}
