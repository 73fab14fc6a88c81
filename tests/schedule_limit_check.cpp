// Host-side check of the work list's limit: build_schedule with a limit gives
// the list it gives without one where that costs the limit or less, and an
// empty one otherwise.  Prints the number of comparisons.
#include <cstdio>

#include "tslb_tiles.h"

using namespace tslb::tile;

static bool same(const Schedule& a, const Schedule& b) {
    if (a.grid != b.grid || a.nseg != b.nseg || a.tz != b.tz || a.split != b.split || a.cost != b.cost ||
        a.seg.size() != b.seg.size())
        return false;
    for (size_t k = 0; k < a.seg.size(); ++k)
        if (a.seg[k].x != b.seg[k].x || a.seg[k].y != b.seg[k].y || a.seg[k].z != b.seg[k].z) return false;
    return true;
}

int main() {
    int n = 0;
    for (int columns : {1, 3, 8, 50, 176, 700})
        for (int nz : {1, 5, 64, 203, 600}) {
            const Schedule s = build_schedule(columns, nz, 256);
            for (long long d : {-1000LL, -3LL, -1LL, 0LL, 1LL, 4LL, 1000LL}) {
                const long long limit = s.cost + d;
                if (limit < 0) continue;
                const Schedule t = build_schedule(columns, nz, 256, limit);
                if (d < 0 ? t.grid != 0 || !t.seg.empty() : !same(s, t)) {
                    printf("FAIL %d %d %lld\n", columns, nz, limit);
                    return 1;
                }
                ++n;
            }
        }
    printf("%d\n", n);
    return 0;
}
