// Tiled update kernel for gfx950: 2.5D z-march with the populations
// exchanged through LDS.
//
// The update of Section 2.2 pulls, for every node x and velocity c, the
// population that the upstream node x - c emits along c, rebuilt from that
// node's moments.  Here every node rebuilds its own 27 emitted populations
// exactly once per step and publishes them in LDS; each node then gathers
// the 27 arriving values from its neighbours.  The arithmetic per
// population is identical to the direct pull, only the sharing differs
// (thread-safe as in the paper: the level-t moments are read-only, the new
// level goes to a separate buffer).
//
// Per node the emitted populations are 216 w(c) P(c) with P a polynomial of
// degree <= 3 in the components of c.  Because c_a^3 = c_a on D3Q27, P has
// 17 monomial coefficients (1, c_a, c_a^2, c_a c_b, c_a^2 c_b, cx cy cz):
// they are formed once per node, the 27 values follow by a separable
// evaluation over z, then x, then y.  The arriving populations are reduced
// to moments by the transposed separable sums.
//
// Tile = TX x TY interior columns plus a one-node halo ring (three more
// waves) marching a segment of planes along z (plus one halo plane each
// side); one resident block per CU walks its list of segments, built on the
// host when the handle is created (tile::build_schedule).  A plane's emitted
// populations with (cx, cy) != (0, 0) go through LDS; the three with
// cx = cy = 0 stay in the thread.  Contributions to the output planes
// p - 1, p, p + 1 are accumulated in three rolling register sets.
//
// What bounds it.  With FP32 storage, memory: on the 512 x 256 x 256 channel
// its counted HBM traffic (1.15 x its algorithmic bytes) moves at 97 % of the
// rate of a plain copy (ten streams in and ten out without arithmetic, in an
// older loop, took 545 us); the arithmetic alone takes 263 us.  With 16-bit
// storage the two are near each other (326 and 275 us).  So the plane loop is
// built to overlap them:
//  - Interior and halo waves run loops of their own (wave-uniform branch), so
//    every wait for memory counts exactly what is in flight.  In one shared
//    loop the waits at the merge points covered loads issued a moment before
//    and the stores of the same plane.
//  - A plane's stores are issued after the next plane's values have arrived
//    (arrive()): loads and stores share one counter that completes in order,
//    so a wait issued after the stores waits for them too.
//  - The halo planes at the ends of a segment, which no output plane belongs
//    to, exchange and sum one of the three cz slices only (64^3 periodic 10.9
//    -> 10.1 us).
// 512 x 256 x 256 channel FP32 559 -> 533 us, FP16 430 -> 392 us; 64^3
// periodic FP32 11.8 -> 10.1 us (all in tiles of 12 rows).
// Tried without gain: two columns of two fields per lane and memory
// instruction for 16-bit storage (sorting them costs what the fewer
// instructions save), two resident blocks of 6 or 7 rows per CU (FP16 485 us
// against 391: more halo columns per node).
#pragma once
#include <type_traits>

#include "tslb_tiles.h"

namespace tslb {
namespace {

using namespace tile;

// Stored values of a node as loaded, one register per field (16-bit storage
// in its lower half).
template <class S>
using raw_t = std::conditional_t<sizeof(typename S::T) == 4, float, unsigned>;
// Loads the ten fields at byte offset `off` of the plane at `plane`;
// consecutive fields are `stride` bytes apart.
template <class S>
__device__ __forceinline__ void load_raw(const char* plane, size_t stride, unsigned off, raw_t<S> (&r)[10]) {
    FieldAddress f(plane, off);
#pragma unroll
    for (int q = 0; q < 10; ++q) {
        if constexpr (sizeof(typename S::T) == 4)
            r[q] = *f.template lane<const float>();
        else
            r[q] = *f.template lane<const unsigned short>();
        f.next(stride);
    }
}

// Converted 16-bit moments of load_raw.  drho and u get their scales; Pi^neq
// is left unscaled: the caller folds 1 / scale[2] into 1 - omega, the only
// factor Pi^neq meets in coefficients() (exact, a power of two).
template <class S>
__device__ __forceinline__ void convert_raw(const raw_t<S> (&r)[10], const StepParams& p, float (&m)[10]) {
#pragma unroll
    for (int q = 0; q < 10; ++q) m[q] = S::convert(__builtin_bit_cast(typename S::T, (unsigned short)r[q]));
    m[0] *= p.inv_scale[0];
#pragma unroll
    for (int q = 1; q < 4; ++q) m[q] *= p.inv_scale[1];
}

// Waits here for the loads into r; 16-bit values are converted into m.
template <class S>
__device__ __forceinline__ void arrive(raw_t<S> (&r)[10], const StepParams& p, float (&m)[10]) {
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (sizeof(typename S::T) == 4) {
        asm volatile("" : "+v"(r[0]), "+v"(r[1]), "+v"(r[2]), "+v"(r[3]), "+v"(r[4]), "+v"(r[5]), "+v"(r[6]), "+v"(r[7]),
                     "+v"(r[8]), "+v"(r[9]));
    } else {
        convert_raw<S>(r, p, m);
        asm volatile("" : "+v"(m[0]), "+v"(m[1]), "+v"(m[2]), "+v"(m[3]), "+v"(m[4]), "+v"(m[5]), "+v"(m[6]), "+v"(m[7]),
                     "+v"(m[8]), "+v"(m[9]));
    }
    __builtin_amdgcn_sched_barrier(0);
}
// The node's moments once they have arrived.
template <class S>
__device__ __forceinline__ const float (&arrived(const raw_t<S> (&r)[10], const float (&m)[10]))[10] {
    if constexpr (sizeof(typename S::T) == 4)
        return r;
    else
        return m;
}

// NT: non-temporal output stores,
// a template parameter since the compiler merges a branch between the two
// kinds into plain stores (4 % slower on the FP32 channels).  XGHOST: grids
// with x ghost faces, whose fluid neighbours also write those ghost nodes.
template <class S, bool WALLS, bool FIELD, int ORDER, int LAT, bool NT, bool XGHOST, bool LATE>
__global__ void __launch_bounds__(NTHREADS, TSLB_WAVES_PER_EU)
    update_tiled_kernel(const char* __restrict__ in, char* __restrict__ out, StepParams p, int tiles_x) {
    static_assert(TX == 64 && 4 + 2 * TY <= 64 && NTHREADS == NINT + 192, "one wave per row, three halo waves");
    __shared__ float lds[NSLOT][LY][LX];
    using T = typename S::T;
    using Raw = raw_t<S>;
    constexpr unsigned kSize = sizeof(T);
    // D3Q27: the populations travel without their weights, which the gather
    // applies for free (add_slice); D3Q19's weights are not separable
    constexpr bool kDeferWeights = LAT == 27;
    // How far loads run ahead.  FP32 with non-temporal stores: two plane-steps,
    // in two register sets used in turn (kTwo).  LATE: to the next plane, with
    // this one's exchange (see loads_late).  Else, 16-bit: one set, converted
    // out of as it arrives and reloaded at once, a whole plane-step ahead.
    constexpr bool kTwo = kSize == 4 && NT, kOne = LATE;
    static_assert(kSize == 2 || NT != LATE);
    // Tiles whose rows are not the frame's (see crosses_up): the rows on both
    // sides of a border of the frame evaluate one slice twice, the halo rows
    // elsewhere theirs in full.  Halo rows collapsed at every tile border were
    // faster with walls (FP16 channels 512 x 256 x 256 378 us, now 389, 384 x
    // 192 x 192 173 and 179) and as fast without (256^3 FP16 189, 187; 64^3
    // FP32 8.9, 9.0), but their values depended on the tile height.
    constexpr bool kOtherRows = kDeferWeights && TY != kFrameY;
    static_assert(TX == kFrameX);
    const Geometry& g = p.geo;
    const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
    const bool pz = (g.periodic & 4) != 0;
    const unsigned plane_nodes = (unsigned)nx * (unsigned)ny;
    const size_t plane_bytes = (size_t)plane_nodes * kSize;
    const size_t stride = (size_t)g.N * kSize;
    // this block's segments (uniform loads); an empty list ends the block
    // before any barrier
    const int4* __restrict__ segs = p.sched + (size_t)blockIdx.x * p.sched_nseg;
    int4 t = segs[0];
    if (t.x < 0) return;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const bool zlo_wall = (g.lo_solid & 4) != 0, zhi_wall = (g.hi_solid & 4) != 0;

    auto in_plane = [&](int z) { return in + plane_bytes * (size_t)z; };
    // 1 - omega of plane z: a scalar load (the table is constant here)
    auto omo_of = [&](int z) {
        return p.omo_z ? reinterpret_cast<const __attribute__((address_space(4))) float*>((uintptr_t)p.omo_z)[z]
                       : p.one_minus_omega;
    };
    auto load_force = [&](unsigned col, int z, float (&gv)[3]) {
        FieldAddress f(reinterpret_cast<const char*>(p.gfield) + (size_t)plane_nodes * 4 * (size_t)z, col * 4u);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            gv[a] = *f.template lane<const float>();
            f.next((size_t)g.N * 4);
        }
    };
    auto force_here = [](float (&gv)[3]) { asm volatile("" : "+v"(gv[0]), "+v"(gv[1]), "+v"(gv[2])); };
    auto solid_col = [&](int wx, int wy) {
        return WALLS && ((wx == 0 && (g.lo_solid & 1)) || (wx == nx - 1 && (g.hi_solid & 1)) ||
                         (wy == 0 && (g.lo_solid & 2)) || (wy == ny - 1 && (g.hi_solid & 2)));
    };
    // Wall nodes emit nothing: their stored moments are the zero deviation
    // (rest state) and their forcing is switched off (gon, and here on wall
    // planes), so every population they publish is exactly 0 and the gather
    // needs no masking.  Fluid neighbours get the bounced-back populations
    // instead.  1 - omega takes the stored Pi^neq scale (see convert_raw).
    auto build = [&](const float (&m)[10], const float (&gv)[3], float gon, int zp, float omo, float A[NK]) {
        float gl[3];
        const float on = WALLS && ((zlo_wall && zp == 0) || (zhi_wall && zp == nz - 1)) ? 0.0f : gon;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const float f = FIELD ? gv[a] : p.force[a];
            gl[a] = WALLS ? on * f : f;
        }
        coefficients<ORDER, LAT>(m, gl, kSize == 4 ? omo : omo * p.inv_scale[2], A);
        // no multiplication of the coefficients is fused into the evaluation
        // that follows, which differs between the roles
        if constexpr (ORDER == 2 && LAT == 27) {
#pragma unroll
            for (int k = K000; k <= K011; ++k) asm volatile("" : "+v"(A[k]));
        }
    };
    if (wave >= NINT / 64) {
        // ------------------------------------------------------- halo waves
        // One kind of column per wave: the row below the tile (what it sends
        // into the tile has cy = +1), the row above (cy = -1), then the four
        // corners and the two side columns (cx = +1 on the left, -1 on the
        // right).
        const int kind = wave - NINT / 64 + 1;
        int lx, ly;  // LDS column and row
        bool publish = true;
        if (kind < 3) {
            lx = 1 + lane;
            ly = kind == 1 ? 0 : LY - 1;
        } else if (lane < 4) {
            lx = (lane & 1) ? LX - 1 : 0;
            ly = (lane & 2) ? LY - 1 : 0;
        } else {
            lx = lane - 4 < TY ? 0 : LX - 1;
            ly = 1 + (lane - 4) % TY;
            publish = lane < 4 + 2 * TY;
        }
        struct Column {
            unsigned node;  // node in plane, wrapped or clamped
            float gon;
            int row;  // the first one above the border of the tile, in the frame's cell (see crosses_up)
        };
        auto column = [&](int col_id) {
            const int y0 = (col_id / tiles_x) * TY;
            const int wx = wrap_or_clamp((col_id % tiles_x) * TX - 1 + lx, nx, g.periodic & 1);
            const int wy = wrap_or_clamp(y0 - 1 + ly, ny, g.periodic & 2);
            return Column{(unsigned)wx + (unsigned)nx * (unsigned)wy, solid_col(wx, wy) ? 0.0f : 1.0f,
                          (kind == 1 ? y0 : y0 + TY) % kFrameY};
        };
        Raw r[10];
        float m[10];
        float gv[3] = {0.0f, 0.0f, 0.0f};
        float omo;
        auto fetch = [&](unsigned node, int z) {
            if constexpr (FIELD) load_force(node, z, gv);
            load_raw<S>(in_plane(z), stride, node * kSize, r);
        };
        auto here = [&] {
            arrive<S>(r, p, m);
            if constexpr (FIELD) force_here(gv);
        };
        Column c = column(t.x);
        {
            const int z = plane_index(t.y - 1, nz, pz);
            fetch(c.node, z);
            omo = omo_of(z);
            here();
        }
        float* const w = &lds[0][ly][lx];
        for (int k = 0;;) {
            const int4 tn = k + 1 < p.sched_nseg ? segs[k + 1] : make_int4(-1, 0, 0, 0);
            const bool more = tn.x >= 0;
            const Column cn = column(more ? tn.x : t.x);
            const int zs = t.y, ze = t.z;
            for (int zp = zs - 1; zp <= ze; ++zp) {
                float A[NK];
                build(arrived<S>(r, m), gv, c.gon, zp, omo, A);
                // The nine populations a halo column sends into the tile: the
                // side columns' and corners' collapsed on x, the rows'
                // collapsed on y at a border of the frame, else in full.
                auto put = [&]<int I>(float v) { w[slot_of(I) * LY * LX] = v; };
                if constexpr (kDeferWeights) {
                    float Q[27];
                    if (kind != 3) {
                        auto rows = [&]<bool COLLAPSED>() {
                            if constexpr (COLLAPSED)
                                collapsed_y(A, kind == 1 ? 1.0f : -1.0f, Q);
                            else
                                populations<27, false>(A, Q);
                            auto value = [&](int I) {
                                return Q[COLLAPSED ? 9 + 3 * (cz_of(I) + 1) + cx_of(I) + 1 : I];
                            };
                            if (kind == 1)
                                Unroll<0, 27>::run([&]<int I>() {
                                    if constexpr (cy_of(I) == 1) put.template operator()<I>(value(I));
                                });
                            else
                                Unroll<0, 27>::run([&]<int I>() {
                                    if constexpr (cy_of(I) == -1) put.template operator()<I>(value(I));
                                });
                        };
                        int row = c.row;
                        if constexpr (kOtherRows) asm volatile("" : "+s"(row));
                        if (!kOtherRows || row == 0)
                            rows.template operator()<true>();
                        else
                            rows.template operator()<false>();
                    } else {
                        collapsed_x(A, lx == 0 ? 1.0f : -1.0f, Q);
                        if (publish && lx == 0)
                            Unroll<0, 27>::run([&]<int I>() {
                                if constexpr (cx_of(I) == 1) put.template operator()<I>(Q[9 + 3 * (cz_of(I) + 1) + cy_of(I) + 1]);
                            });
                        if (publish && lx != 0)
                            Unroll<0, 27>::run([&]<int I>() {
                                if constexpr (cx_of(I) == -1) put.template operator()<I>(Q[9 + 3 * (cz_of(I) + 1) + cy_of(I) + 1]);
                            });
                    }
                } else {
                    float G[27];
                    populations<LAT, true>(A, G);
                    if (publish)
                        Unroll<0, 27>::run([&]<int I>() {
                            if constexpr ((cx_of(I) != 0 || cy_of(I) != 0) && carries<LAT>(I)) put.template operator()<I>(G[I]);
                        });
                }
                const bool on = zp + 1 <= ze;
                const int z = plane_index(on ? zp + 1 : (more ? tn.y - 1 : ze), nz, pz);
                const unsigned node = on ? c.node : cn.node;
                // With kTwo, loads before the exchange: the interior waves of
                // the neighbouring tile have asked for these lines a plane
                // earlier.  Otherwise after it, when those have just asked
                // (512 x 256 x 256 channel FP16 393 us against 440; FP32 553
                // against 533; 181 x 428 x 145 FP32 212 against 229).
                if constexpr (kTwo) fetch(node, z);
                __syncthreads();
                if constexpr (!kTwo) fetch(node, z);
                omo = omo_of(z);
                __syncthreads();
                here();
            }
            if (!more) return;
            ++k;
            t = tn;
            c = cn;
        }
    }

    // ---------------------------------------------------------- interior waves
    const int ly = 1 + wave;
    const int lx = 1 + lane;
    struct Column {
        int gx, gy;     // grid coordinates (beyond the grid in its last tiles)
        unsigned node;  // node in plane, wrapped or clamped
        float gon;
    };
    auto column = [&](int col_id) {
        Column c;
        c.gx = (col_id % tiles_x) * TX + lane;
        c.gy = (col_id / tiles_x) * TY + wave;
        const int wx = wrap_or_clamp(c.gx, nx, g.periodic & 1);
        const int wy = wrap_or_clamp(c.gy, ny, g.periodic & 2);
        c.node = (unsigned)wx + (unsigned)nx * (unsigned)wy;
        c.gon = solid_col(wx, wy) ? 0.0f : 1.0f;
        return c;
    };

    Raw rcur[10], rnx[10];
    float m[10];
    float gv[3] = {0.0f, 0.0f, 0.0f};
    float omo;
    Column c = column(t.x);
    {
        const int z = plane_index(t.y - 1, nz, pz);
        if constexpr (FIELD) load_force(c.node, z, gv);
        load_raw<S>(in_plane(z), stride, c.node * kSize, rcur);
        if constexpr (kTwo) load_raw<S>(in_plane(plane_index(t.y, nz, pz)), stride, c.node * kSize, rnx);
        omo = omo_of(z);
        arrive<S>(rcur, p, m);
        if constexpr (FIELD) force_here(gv);
    }
    for (int k = 0;;) {
        // the block's next segment: its first planes are loaded during the
        // last planes of this one
        const int4 tn = k + 1 < p.sched_nseg ? segs[k + 1] : make_int4(-1, 0, 0, 0);
        const bool more = tn.x >= 0;
        const Column cn = column(more ? tn.x : t.x);
        const int gx = c.gx, gy = c.gy, zs = t.y, ze = t.z;
        // rows are uniform over a wave: walls and ghosts on y are scalar
        const bool row_fluid = gy < ny && !(gy == 0 && ((g.lo_solid | g.lo_ghost) & 2)) &&
                               !(gy == ny - 1 && ((g.hi_solid | g.hi_ghost) & 2));
        const bool col_fluid = row_fluid && gx < nx && !(gx == 0 && ((g.lo_solid | g.lo_ghost) & 1)) &&
                               !(gx == nx - 1 && ((g.hi_solid | g.hi_ghost) & 1));
        // do this row's populations with cy = +1 (-1) cross a border of the frame?
        const int frame_row = gy % kFrameY;
        const bool xwalls = WALLS && ((g.lo_solid | g.hi_solid) & 1) != 0;
        const bool ylo = WALLS && (g.lo_solid & 2) && gy == 1, yhi = WALLS && (g.hi_solid & 2) && gy == ny - 2;
        const bool xlo = WALLS && (g.lo_solid & 1) && gx == 1, xhi = WALLS && (g.hi_solid & 1) && gx == nx - 2;
        // One plane zp: build and publish its populations, add what arrives
        // from it to the output planes zp - 1 (aprev), zp (acur) and zp + 1
        // (anext, which starts here), then store the completed plane zp - 1.
        // The halo planes at the two ends of the segment contribute one slice
        // only: PART 1 (first, zs - 1) cz = +1 to the plane above, PART 2
        // (last, ze) cz = -1 to the plane below, a third of the exchange and
        // about half the arithmetic of a plane.
        auto plane = [&]<int BUF, int PART>(int zp, MomentSums& aprev, MomentSums& acur, MomentSums& anext) {
            // is velocity I part of this plane's exchange?
            constexpr auto moves = [](int I) { return carries<LAT>(I) && (PART == 0 || cz_of(I) == (PART == 1 ? 1 : -1)); };
            // the plane after this one, of this segment or the next; loads
            // past the last segment repeat its last plane
            const bool on = zp + 1 <= ze;
            const int z1 = plane_index(on ? zp + 1 : (more ? tn.y - 1 : ze), nz, pz);
            if constexpr (!kTwo && !kOne) load_raw<S>(in_plane(z1), stride, (on ? c.node : cn.node) * kSize, rcur);
            const float omo1 = omo_of(z1);
            // (compared here: kept as masks across the planes they spill)
            int row = frame_row;
            if constexpr (kOtherRows) asm volatile("" : "+s"(row));
            const bool up = kOtherRows && row == kFrameY - 1, down = kOtherRows && row == 0;
            float G[27];
            {
                float A[NK];
                if constexpr (kTwo && BUF == 1)
                    build(arrived<S>(rnx, m), gv, c.gon, zp, omo, A);
                else
                    build(arrived<S>(rcur, m), gv, c.gon, zp, omo, A);
                populations<LAT, !kDeferWeights>(A, G);
                if constexpr (kOtherRows) {
                    // the buffer is free since the previous plane's second barrier
                    auto collapsed_row = [&]<int CY>() {
                        float Q[27];
                        collapsed_y(A, CY, Q);
                        Unroll<0, 27>::run([&]<int I>() {
                            if constexpr (cy_of(I) == CY && moves(I))
                                lds[slot_of(I)][ly][lx] = Q[9 + 3 * (cz_of(I) + 1) + cx_of(I) + 1];
                        });
                    };
                    if (up) collapsed_row.template operator()<1>();
                    if (down) collapsed_row.template operator()<-1>();
                }
            }
            // the value that stays is rounded with its weight 12, like those
            // that go through LDS
            if constexpr (LAT == 19) asm volatile("" : "+v"(G[13]));
            if constexpr (WALLS && PART == 0) {
                // half-way bounce-back in place: a fluid node next to a wall
                // receives its own population along -c for every c whose
                // upstream node is solid; it holds those values right here
                const bool zlo = zlo_wall && zp == 1, zhi = zhi_wall && zp == nz - 2;
                if ((ylo || yhi || zlo || zhi || xwalls) && col_fluid) {
                    Unroll<0, 27>::run([&]<int I>() {
                        constexpr int X = cx_of(I), Y = cy_of(I), Z = cz_of(I);
                        bool s = false;
                        if (Y == 1) s |= ylo;
                        if (Y == -1) s |= yhi;
                        if (Z == 1) s |= zlo;
                        if (Z == -1) s |= zhi;
                        if (X == 1) s |= xlo;
                        if (X == -1) s |= xhi;
                        if constexpr (carries<LAT>(I))
                            if (s) acur.template add<I>(kDeferWeights ? w216_of(I) * G[26 - I] : G[26 - I]);
                    });
                }
            }
            auto publish = [&]<int CY>() {
                Unroll<0, 27>::run([&]<int I>() {
                    if constexpr (cy_of(I) == CY && (cx_of(I) != 0 || CY != 0) && moves(I)) lds[slot_of(I)][ly][lx] = G[I];
                });
            };
            if (!down) publish.template operator()<-1>();
            publish.template operator()<0>();
            if (!up) publish.template operator()<1>();
            if constexpr (FIELD) load_force(on ? c.node : cn.node, z1, gv);
            if constexpr (kOne) load_raw<S>(in_plane(z1), stride, (on ? c.node : cn.node) * kSize, rcur);
            if constexpr (kTwo) {
                // this plane's set is free again: the plane after next
                const bool on2 = zp + 2 <= ze;
                const int z2 = plane_index(on2 ? zp + 2 : (!more ? ze : (zp + 2 == ze + 1 ? tn.y - 1 : tn.y)), nz, pz);
                if constexpr (BUF == 1)
                    load_raw<S>(in_plane(z2), stride, (on2 ? c.node : cn.node) * kSize, rnx);
                else
                    load_raw<S>(in_plane(z2), stride, (on2 ? c.node : cn.node) * kSize, rcur);
            }
            __syncthreads();
            // the values arriving through LDS go to registers at once, so the
            // buffer is free again after the second barrier and the sums, the
            // stores and the next plane's build form one barrier-free phase
            float F[3][3][3];  // [cz + 1][cy + 1][cx + 1]
            Unroll<0, 27>::run([&]<int I>() {
                constexpr int X = cx_of(I), Y = cy_of(I), Z = cz_of(I);
                if constexpr (X == 0 && Y == 0)
                    F[Z + 1][1][1] = G[I];
                else if constexpr (!moves(I))
                    F[Z + 1][Y + 1][X + 1] = 0.0f;
                else
                    F[Z + 1][Y + 1][X + 1] = lds[slot_of(I)][ly - Y][lx - X];
            });
            __syncthreads();
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (PART != 1) add_slice<-1, false, kDeferWeights>(F[0], aprev);
            if constexpr (PART == 0) add_slice<0, false, kDeferWeights>(F[1], acur);
            if constexpr (PART != 2) add_slice<1, true, kDeferWeights>(F[2], anext);
            // before the stores: a wait after them would wait for those too
            if constexpr (kTwo && BUF == 0)
                arrive<S>(rnx, p, m);
            else
                arrive<S>(rcur, p, m);
            if constexpr (FIELD) force_here(gv);
            omo = omo1;
            if constexpr (PART == 1) return;
            const int zo = zp - 1;
            if (zo >= zs && !(zo == 0 && ((g.lo_solid | g.lo_ghost) & 4)) &&
                !(zo == nz - 1 && ((g.hi_solid | g.hi_ghost) & 4)) && col_fluid) {
                float o[10];
                if constexpr (kSize == 4)
                    finalize<LAT == 19 ? 36 : 216>(aprev, o);
                else
                    finalize_unscaled<LAT == 19 ? 36 : 216>(aprev, o);
                // 16-bit storage: 1 / 216 and the field's scale in one factor
                constexpr float kInv = 1.0f / (LAT == 19 ? 36.0f : 216.0f);
                const float k0 = kInv * p.scale[0], k1 = p.scale[1], k2 = kInv * p.scale[2];
                auto factor = [&](int q) { return q == 0 ? k0 : q < 4 ? k1 : k2; };
                char* const b0 = out + plane_bytes * (size_t)zo;
                auto put = [&](unsigned off) {
                    FieldAddress f(b0, off);
#pragma unroll
                    for (int q = 0; q < 10; ++q) {
                        store_out<NT>(f.template lane<store_bits<T>>(),
                                      __builtin_bit_cast(store_bits<T>, S::pack(kSize == 4 ? o[q] : factor(q) * o[q])));
                        f.next(stride);
                    }
                };
                const unsigned on_bytes = c.node * kSize;
                put(on_bytes);
                if constexpr (XGHOST) {
                    // A ghost node of an x face next to this fluid node
                    // takes its values (Section 2.3 refill; an inlet's
                    // velocity is imposed by the refill pass): stored here,
                    // into the cache line this row's stores fill anyway.
                    // This node is fluid, so that ghost lies on no other
                    // ghost face.
                    if ((g.lo_ghost & 1) && gx == 1) put(on_bytes - kSize);
                    if ((g.hi_ghost & 1) && gx == nx - 2) put(on_bytes + kSize);
                }
            }
        };

        // Rolling roles of the three accumulators, unrolled to their period
        // (and that of the two register sets) so every role is fixed.
        MomentSums a0, a1, a2, done;  // done: plane ze - 1 before its last slice
        a1.zero();
        plane.template operator()<0, 1>(zs - 1, a0, a1, a2);
        if constexpr (kTwo) {
            for (int zp = zs;; zp += 6) {
                plane.template operator()<1, 0>(zp, a1, a2, a0);
                done = a2;
                if (zp + 1 == ze) break;
                plane.template operator()<0, 0>(zp + 1, a2, a0, a1);
                done = a0;
                if (zp + 2 == ze) break;
                plane.template operator()<1, 0>(zp + 2, a0, a1, a2);
                done = a1;
                if (zp + 3 == ze) break;
                plane.template operator()<0, 0>(zp + 3, a1, a2, a0);
                done = a2;
                if (zp + 4 == ze) break;
                plane.template operator()<1, 0>(zp + 4, a2, a0, a1);
                done = a0;
                if (zp + 5 == ze) break;
                plane.template operator()<0, 0>(zp + 5, a0, a1, a2);
                done = a1;
                if (zp + 6 == ze) break;
            }
            if (((ze - zs) & 1) == 0) {
                plane.template operator()<1, 2>(ze, done, a0, a1);
            } else {
                plane.template operator()<0, 2>(ze, done, a0, a1);
                // an odd number of steps left the next segment's first plane
                // in rnx: swap the sets so that it starts on rcur again
#pragma unroll
                for (int q = 0; q < 10; ++q) {
                    const Raw v = rcur[q];
                    rcur[q] = rnx[q];
                    rnx[q] = v;
                }
            }
        } else {
            for (int zp = zs;; zp += 3) {
                plane.template operator()<0, 0>(zp, a1, a2, a0);
                done = a2;
                if (zp + 1 == ze) break;
                plane.template operator()<0, 0>(zp + 1, a2, a0, a1);
                done = a0;
                if (zp + 2 == ze) break;
                plane.template operator()<0, 0>(zp + 2, a0, a1, a2);
                done = a1;
                if (zp + 3 == ze) break;
            }
            plane.template operator()<0, 2>(ze, done, a0, a1);
        }
        if (!more) return;
        ++k;
        t = tn;
        c = cn;
    }
}

// Tile columns of a grid.
inline int tile_columns(const Geometry& g) { return ((g.n[0] + TX - 1) / TX) * ((g.n[1] + TY - 1) / TY); }

template <class S>
bool rows_whole_lines(const StepParams& p) {
    return ((long long)p.geo.n[0] * (long long)sizeof(typename S::T)) % 128 == 0;
}
inline bool x_ghost_faces(const StepParams& p) { return ((p.geo.lo_ghost | p.geo.hi_ghost) & 1) != 0; }
// Does the update write the x-face ghost nodes next to fluid nodes (XGHOST)?
// It pays on rows of whole cache lines, where the ghost shares its
// neighbour's line; grids with walls or a force field have no such variant.
template <class S>
bool writes_x_ghosts(const StepParams& p) {
    return x_ghost_faces(p) && (p.geo.lo_solid | p.geo.hi_solid) == 0 && p.gfield == nullptr && rows_whole_lines<S>(p);
}

template <class S, bool WALLS, bool FIELD, int ORDER, int LAT, bool NT, bool XGHOST, bool LATE = sizeof(typename S::T) == 4 && !NT>
hipError_t launch_k(const void* in, void* out, const StepParams& p, hipStream_t s) {
    if (p.geo.N >= (1LL << 30)) return hipErrorInvalidValue;  // 32-bit byte offsets
    if (!p.sched || p.sched_grid < 8 || p.sched_nseg < 1) return hipErrorInvalidValue;
    const int tiles_x = (p.geo.n[0] + TX - 1) / TX;
    hipLaunchKernelGGL((update_tiled_kernel<S, WALLS, FIELD, ORDER, LAT, NT, XGHOST, LATE>), dim3(p.sched_grid),
                       dim3(NTHREADS), 0, s, (const char*)in, (char*)out, p, tiles_x);
    return hipGetLastError();
}

// Non-temporal output stores when every row starts on a cache line (the new
// level is not read again by this launch); otherwise plain ones, so that L2
// merges the lines that neighbouring tiles share (see store_out).  Plain ones
// also where the two FP32 levels fit the Infinity Cache, in which the next
// step then finds its input (non-temporal / plain: 128^3 channel, 168 MB, 44.9
// / 34.6 us; 192 x 128 x 128, 252 MB, 63.2 / 53.1; 160^3 channel, 328 MB, 78.5
// / 78.9).  16-bit levels, bound by arithmetic there, stay non-temporal (128^3
// FP16 33.4 / 34.4).
template <class S>
bool streams_out(const StepParams& p) {
    constexpr size_t kSize = sizeof(typename S::T);
    return rows_whole_lines<S>(p) && (kSize == 2 || 20 * kSize * (size_t)p.geo.N > kInfinityCacheBytes);
}

// Loads with the exchange (LATE)?  Where tiles share lines, two planes of all
// blocks of an XCD push the halves of stored lines out of its L2 before the
// neighbour completes them, so the loads run ahead less: FP32 on every such
// grid (us, two planes ahead / late: 333 x 101 x 77 45.0 / 44.5, 181 x 428 x
// 145 220 / 212); 16-bit D3Q27 in tiles of 12 rows, without walls or a force
// field, where two levels stay about in the Infinity Cache (us, a plane ahead /
// late: 110 x 131 x 313 FP16 64.8 / 61.4, 271 x 271 x 39 46.5 / 44.1, 160 x 200
// x 210, 269 MB, 89.2 / 86.5, 77 x 300 x 300, 277 MB, 126.3 / 124.3; beyond, 129
// x 400 x 140, 289 MB, 121.1 / 124.7, 250^3 196.1 / 203.5; with a field 160 x
// 992 x 32 66.5 / 70.9; 13 rows 333 x 210 x 140 137 / 143.6; walls and D3Q19
// gain 2 to 5 % from it, but are faster than before without).
template <class S>
bool loads_late(const StepParams& p) {
    return !rows_whole_lines<S>(p) && 40 * (size_t)p.geo.N <= kInfinityCacheBytes / 20 * 21;
}

template <class S, bool WALLS, bool FIELD, int ORDER, int LAT>
hipError_t launch_t(const void* in, void* out, const StepParams& p, hipStream_t s) {
    const bool nt = streams_out<S>(p);
    if constexpr (!WALLS && !FIELD)
        if (writes_x_ghosts<S>(p)) {
            if constexpr (sizeof(typename S::T) == 4)
                if (!nt) return launch_k<S, false, false, ORDER, LAT, false, true>(in, out, p, s);
            return launch_k<S, false, false, ORDER, LAT, true, true>(in, out, p, s);
        }
    if (nt) return launch_k<S, WALLS, FIELD, ORDER, LAT, true, false>(in, out, p, s);
    if constexpr (sizeof(typename S::T) == 2 && TY == kFrameY && !FIELD && !WALLS && LAT == 27)
        if (loads_late<S>(p)) return launch_k<S, WALLS, FIELD, ORDER, LAT, false, false, true>(in, out, p, s);
    return launch_k<S, WALLS, FIELD, ORDER, LAT, false, false>(in, out, p, s);
}

template <class S, int ORDER, int LAT>
hipError_t launch_o(const void* in, void* out, const StepParams& p, hipStream_t s) {
    const bool walls = (p.geo.lo_solid | p.geo.hi_solid) != 0;
    const bool field = p.gfield != nullptr;
    if (walls)
        return field ? launch_t<S, true, true, ORDER, LAT>(in, out, p, s)
                     : launch_t<S, true, false, ORDER, LAT>(in, out, p, s);
    return field ? launch_t<S, false, true, ORDER, LAT>(in, out, p, s)
                 : launch_t<S, false, false, ORDER, LAT>(in, out, p, s);
}

template <class S>
hipError_t launch_s(const void* in, void* out, const StepParams& p, hipStream_t s) {
    if (p.lattice == 19)
        return p.order == 2 ? launch_o<S, 2, 19>(in, out, p, s) : launch_o<S, 3, 19>(in, out, p, s);
    return p.order == 2 ? launch_o<S, 2, 27>(in, out, p, s) : launch_o<S, 3, 27>(in, out, p, s);
}

}  // namespace
}  // namespace tslb
