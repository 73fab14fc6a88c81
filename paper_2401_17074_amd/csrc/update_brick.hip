// Brick update kernel for gfx950: the FP32 update of small and narrow grids.
//
// The tiled update marches 64 x 12 columns along z, a plane per step; on a
// grid of a few hundred thousand nodes most of its time is the chain of those
// steps (load, build, exchange, sum: more than a microsecond each) on too few
// blocks.  Here one block updates a brick of BX x BY x BZ nodes at once: four
// waves hold its nodes, seven more its one-node halo; each thread builds its
// node's populations (a halo node the nine that can enter the brick) and
// publishes them in LDS, and after one barrier the four waves gather the
// arriving values of their nodes, sum and store.  One load latency, one
// exchange, no serial chain; the price is 648 nodes built for 256 updated,
// which is why the marching kernel takes over on larger and wider grids (see
// prefers_brick).
#include "tslb_tiles.h"

namespace tslb {
namespace {

using namespace tile;

constexpr int BX = kBrickX, BY = kBrickY, BZ = kBrickZ;
constexpr int HX = BX + 2, HY = BY + 2, HZ = BZ + 2;
constexpr int kBrickNodes = HX * HY * HZ;  // with the halo
constexpr int kBrickOut = BX * BY * BZ;
// 4 waves of the brick's nodes, 2 of the z faces, 2 of the y faces, 1 of the
// four edges along x, 2 of the x faces with all their edges and corners
static_assert(kBrickThreads == kBrickOut + 2 * 64 + 2 * 64 + 64 + 128);
static_assert(BX * BY == 64 && BX * BZ == 64 && 4 * BX == 64 && 2 * HY * HZ <= 128, "whole wavefronts per role");
static_assert(27 * kBrickNodes * 4 * 2 <= 163840, "two bricks per CU");

// In-range index of coordinate v >= -1 (periodic axes wrap, others clamp;
// clamped values are never used by a fluid node).
__device__ __forceinline__ int brick_index(int v, int n, bool periodic) {
    if (!periodic) return min(max(v, 0), n - 1);
    if (v < 0) v += n;
    while (v >= n) v -= n;  // once, or more on an axis shorter than a brick
    return v;
}

template <bool WALLS, int ORDER, int LAT>
__global__ void __launch_bounds__(kBrickThreads, 6)
    update_brick_kernel(const float* __restrict__ in, float* __restrict__ out, StepParams p, int bricks_x, int bricks_y,
                        int bricks) {
    constexpr bool kDeferWeights = LAT == 27;
    __shared__ float lds[27][kBrickNodes];
    const Geometry& g = p.geo;
    const size_t stride = (size_t)g.N * 4;
    // each XCD takes a contiguous run of bricks (block ids go round-robin)
    const int per = (int)(gridDim.x >> 3);
    const int b = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
    if (b >= bricks) return;  // padding block, before the barrier
    const int x0 = b % bricks_x * BX, y0 = b / bricks_x % bricks_y * BY, z0 = b / (bricks_x * bricks_y) * BZ;
    const int tid = threadIdx.x;

    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // Coordinates in the brick with its halo, and what of the node's
    // populations is published: all (its own nodes), or the nine with one
    // component fixed, evaluated in full or collapsed as the frame of the
    // evaluation has it (see crosses_up; its borders are borders of bricks).
    enum { kNode, kFullX, kFullY, kFullZ, kX, kY };
    static_assert(kFrameX % BX == 0 && kFrameY % BY == 0, "bricks lie within cells of the frame");
    const bool ylo_frame = crosses_up(y0 - 1, kFrameY), yhi_frame = crosses_down(y0 + BY, kFrameY);
    int hx, hy, hz, role = kNode;
    bool on = true;
    if (wave < 4) {
        hx = 1 + (lane & (BX - 1));
        hy = 1 + lane / BX;
        hz = 1 + wave;
    } else if (wave < 6) {
        role = kFullZ;
        hx = 1 + (lane & (BX - 1));
        hy = 1 + lane / BX;
        hz = wave == 4 ? 0 : HZ - 1;
    } else if (wave < 8) {
        hx = 1 + (lane & (BX - 1));
        hy = wave == 6 ? 0 : HY - 1;
        hz = 1 + lane / BX;
        role = (wave == 6 ? ylo_frame : yhi_frame) ? kY : kFullY;
    } else if (wave == 8) {  // the edges along x
        hx = 1 + (lane & (BX - 1));
        hy = (lane & BX) ? HY - 1 : 0;
        hz = (lane & (2 * BX)) ? HZ - 1 : 0;
        role = (hy == 0 ? ylo_frame : yhi_frame) ? kY : kFullZ;
    } else {
        const int k = (wave - 9) * 64 + lane;  // 36 nodes at each end
        on = k < 2 * HY * HZ;
        hx = k < HY * HZ ? 0 : HX - 1;
        hy = k % HY;
        hz = k / HY % HZ;
        const bool xf = hx == 0 ? crosses_up(x0 - 1, kFrameX) : crosses_down(x0 + BX, kFrameX);
        const bool yf = (hy == 0 && ylo_frame) || (hy == HY - 1 && yhi_frame);
        role = xf ? kX : yf ? kY : kFullX;
    }
    float G[27];
    const int x = x0 - 1 + hx, y = y0 - 1 + hy, z = z0 - 1 + hz;
    const int own = hx + HX * (hy + HY * hz);
    if (on) {
        const int wx = brick_index(x, g.n[0], g.periodic & 1);
        const int wy = brick_index(y, g.n[1], g.periodic & 2);
        const int wz = brick_index(z, g.n[2], g.periodic & 4);
        const unsigned n = (unsigned)wx + (unsigned)g.n[0] * ((unsigned)wy + (unsigned)g.n[1] * (unsigned)wz);
        float m[10];
        FieldAddress f(in, n * 4u);
#pragma unroll
        for (int q = 0; q < 10; ++q) {
            m[q] = *f.template lane<const float>();
            f.next(stride);
        }
        float gl[3] = {p.force[0], p.force[1], p.force[2]};
        if (p.gfield) {
#pragma unroll
            for (int a = 0; a < 3; ++a) gl[a] = p.gfield[(size_t)a * g.N + n];
        }
        // wall nodes emit nothing: they hold the rest state, and no force
        if (WALLS && is_solid(g, wx, wy, wz)) gl[0] = gl[1] = gl[2] = 0.0f;
        float A[NK];
        coefficients<ORDER, LAT>(m, gl, omo_at(p, wz), A);
        float* const w = &lds[0][own];
        if constexpr (LAT == 19) {
            // evaluated in full by every node, as in the tiled update
            populations<19, true>(A, G);
            // the value that stays is rounded with its weight 12 (see there)
            asm volatile("" : "+v"(G[13]));
            Unroll<0, 27>::run([&]<int I>() {
                if constexpr (carries<19>(I) && I != 13) w[I * kBrickNodes] = G[I];
            });
        } else {
            // no multiplication of the coefficients is fused into the
            // evaluation that follows, which differs between the roles
            if constexpr (ORDER == 2) {
#pragma unroll
                for (int k = K000; k <= K011; ++k) asm volatile("" : "+v"(A[k]));
            }
            // the nine populations with component D (0 x, 1 y, 2 z) positive
            // where `low`, negative otherwise; value(I) of the velocity I
            auto put = [&]<int D>(bool low, auto&& value) {
                constexpr int kStep[3] = {1, 3, 9};
                float* const base = w + (low ? 2 * kStep[D] : 0) * kBrickNodes;
                Unroll<0, 27>::run([&]<int I>() {
                    constexpr int c[3] = {cx_of(I), cy_of(I), cz_of(I)};
                    if constexpr (c[D] == -1) base[I * kBrickNodes] = value.template operator()<I, I + 2 * kStep[D]>();
                });
            };
            float Q[27];
            if (role == kNode || role == kFullX || role == kFullY) {
                populations<27, false>(A, G);
                if (role == kNode)
                    Unroll<0, 27>::run([&]<int I>() {
                        if constexpr (I != 13) w[I * kBrickNodes] = G[I];
                    });
                else if (role == kFullX)
                    put.template operator()<0>(hx == 0, [&]<int M, int P>() { return hx == 0 ? G[P] : G[M]; });
                else
                    put.template operator()<1>(hy == 0, [&]<int M, int P>() { return hy == 0 ? G[P] : G[M]; });
            } else if (role == kFullZ) {
                // the slice cz = s of populations()
                const float s = hz == 0 ? 1.0f : -1.0f;
                eval_slice<1, 27, false>(fmaf(s, A[K001], A[K000] + A[K002]), fmaf(s, A[K101], A[K100] + A[K102]),
                                         fmaf(s, A[K011], A[K010] + A[K012]), fmaf(s, A[K201], A[K200]),
                                         fmaf(s, A[K021], A[K020]), fmaf(s, A[K111], A[K110]), A[K210], A[K120], Q);
                put.template operator()<2>(hz == 0, [&]<int M, int P>() { return Q[P]; });
            } else if (role == kY) {
                collapsed_y(A, hy == 0 ? 1.0f : -1.0f, Q);
                put.template operator()<1>(hy == 0, [&]<int M, int P>() { return Q[9 + 3 * (cz_of(M) + 1) + cx_of(M) + 1]; });
            } else {
                collapsed_x(A, hx == 0 ? 1.0f : -1.0f, Q);
                put.template operator()<0>(hx == 0, [&]<int M, int P>() { return Q[9 + 3 * (cz_of(M) + 1) + cy_of(M) + 1]; });
            }
        }
    }
    __syncthreads();
    if (role != kNode) return;
    if (x >= g.n[0] || y >= g.n[1] || z >= g.n[2] || !is_fluid(g, x, y, z)) return;
    const int wf = WALLS ? wall_flags(g, x, y) : 0;
    const bool zlo = WALLS && (g.lo_solid & 4) && z == 1, zhi = WALLS && (g.hi_solid & 4) && z == g.n[2] - 2;
    float F[3][3][3];  // [cz + 1][cy + 1][cx + 1]
    Unroll<0, 27>::run([&]<int I>() {
        constexpr int X = cx_of(I), Y = cy_of(I), Z = cz_of(I);
        if constexpr (!carries<LAT>(I))
            F[Z + 1][Y + 1][X + 1] = 0.0f;
        else if constexpr (I == 13)
            F[1][1][1] = G[13];
        else
            F[Z + 1][Y + 1][X + 1] = lds[I][own - X - HX * (Y + HY * Z)];
    });
    MomentSums a;
    add_slice<1, true, kDeferWeights>(F[2], a);
    if (WALLS && (wf != 0 || zlo || zhi)) {
        // half-way bounce-back: the node's own population along -c comes back
        // where the upstream node is a wall (of equal weight), whose own are
        // zero; added where the tiled update adds them
        Unroll<0, 27>::run([&]<int I>() {
            if constexpr (carries<LAT>(I))
                if (upstream_solid<I>(wf, zlo, zhi)) a.template add<I>(kDeferWeights ? w216_of(I) * G[26 - I] : G[26 - I]);
        });
    }
    add_slice<0, false, kDeferWeights>(F[1], a);
    add_slice<-1, false, kDeferWeights>(F[0], a);
    float o[10];
    finalize<LAT == 19 ? 36 : 216>(a, o);
    const unsigned n = (unsigned)x + (unsigned)g.n[0] * ((unsigned)y + (unsigned)g.n[1] * (unsigned)z);
    FieldAddress f(out, n * 4u);
#pragma unroll
    for (int q = 0; q < 10; ++q) {
        *f.template lane<float>() = o[q];
        f.next(stride);
    }
}

template <bool WALLS, int ORDER, int LAT>
hipError_t launch_k(const float* in, float* out, const StepParams& p, hipStream_t s) {
    const int bx = (p.geo.n[0] + BX - 1) / BX, by = (p.geo.n[1] + BY - 1) / BY;
    const long long bricks = brick_count(p.geo);
    if (p.geo.N >= (1LL << 30) || bricks > kMaxBricks) return hipErrorInvalidValue;
    const unsigned grid = (unsigned)((bricks + 7) & ~7LL);  // whole runs per XCD
    hipLaunchKernelGGL((update_brick_kernel<WALLS, ORDER, LAT>), dim3(grid), dim3(kBrickThreads), 0, s, in, out, p, bx, by,
                       (int)bricks);
    return hipGetLastError();
}

template <int ORDER, int LAT>
hipError_t launch_w(const float* in, float* out, const StepParams& p, hipStream_t s) {
    return (p.geo.lo_solid | p.geo.hi_solid) != 0 ? launch_k<true, ORDER, LAT>(in, out, p, s)
                                                  : launch_k<false, ORDER, LAT>(in, out, p, s);
}

}  // namespace

// Bricks run in rounds of one per CU (two at a time): about 5 us for one and
// 1.8 us for each further one (2.3 where two levels exceed the Infinity Cache,
// for the halo's traffic).  The tiled update takes about 5 us and, with tiles
// of 8 rows, 1.4 us for each plane-step of its longest block, with 12 rows 1.7
// (its list's cost in steps).  us per step of FP32 grids, tiles / bricks
// (rounds, steps):
//   8 rows: 32^3 6.7 / 5.1 (1, 3), 48^3 8.2 / 6.5 (2, 3), 96 x 32 x 32 7.4 / 6.6
//   (2, 3), 64 x 4 x 1024 10.9 / 10.9 (4, 6), 48 x 4 x 8192 44.7 / 47.1 (24, 34),
//   52^3 8.6 / 9.3 (3, 4), 64 x 4 x 12000 63 / 90 (47, 49; 86 in tiles of 12
//   rows), 16 x 4 x 262144 1342 / 589 (256, 1056);
//   12 rows: 16 x 200 x 256 36.2 / 27.1 (13, 20), 8 x 500 x 500 146 / 115 (62,
//   88), 17 x 100 x 100 13.9 / 11.8 (5, 6);
//   12 rows, beyond the cache: 16 x 64 x 16384 670 / 626 (256, 396), 2 x 4096 x
//   2048 4517 / 4003 (2048, 2826), 16 x 2000 x 2000 2301 / 2334 (977, 1355).
// The values do not depend on the choice (see crosses_up).  FP32 only: 16-bit
// grids were not moved to bricks.
bool prefers_brick(int storage, const Geometry& g, long long steps, bool rows8) {
    return brick_grid(storage, g, steps, rows8, compute_units());
}

hipError_t launch_update_brick(const void* in_, void* out_, const StepParams& p, hipStream_t s) {
    const float* in = (const float*)in_;
    float* out = (float*)out_;
    if (p.lattice == 19) return p.order == 2 ? launch_w<2, 19>(in, out, p, s) : launch_w<3, 19>(in, out, p, s);
    return p.order == 2 ? launch_w<2, 27>(in, out, p, s) : launch_w<3, 27>(in, out, p, s);
}

}  // namespace tslb
