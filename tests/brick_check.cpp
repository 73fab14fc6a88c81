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
        const int columns = ((g.n[0] + TX - 1) / TX) * ((g.n[1] + TY - 1) / TY);
        const Schedule s = build_schedule(columns, g.n[2], 256);
        printf("%d %d %d %lld %d %d\n", g.n[0], g.n[1], g.n[2], brick_count(g), (int)brick_grid(0, g, s.cost, 256),
               (int)brick_grid(1, g, s.cost, 256));
    }
    return 0;
}
