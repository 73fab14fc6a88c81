// Tiled discrete adjoint of the update for gfx950: the exact transpose of the
// tiled forward kernel.
//
// Forward: node y emits f_i(y) = w_i P_y(c_i) (P polynomial in c with the 17
// coefficients A_k(M_y, g_y)) to x = y + c_i, and x sums what arrives into
// its new moments M'(x).  Reverse, for a sensitivity lam' = dL/dM'(x):
//   a_x(c) = dL/df_i at x = lam'_rho + lam'_u.(c - u')/rho'
//            + lam'_Pi : [(c - u')(c - u') - delta/3]
// is a quadratic in c (10 coefficients), so every node x evaluates its 27
// arrival sensitivities once and publishes them in LDS; every source node y
// gathers a_{y+c_i}(c_i) from its downstream neighbours, forms the 17
// weighted monomial moments Lambda_k = sum_i w_i m_k(c_i) a_{y+c_i}(c_i), and
// pulls them back through the coefficient map (coefficients_vjp).  Wall
// nodes carry zero sensitivity; a node whose upstream node along c_j is a
// wall received its own population along -c_j there, so a_y(c_j) is added
// as a value arriving along -c_j (done in the same pass for the few lanes
// next to a wall).
//
// Tile, work list, wave roles and thin halo planes are the tiled update's.
// What bounds it: memory, 34 streams of one field each (14 in at t + 1, 10 in
// at t, 10 out; 9 more with a force field and its gradient).  256^3: 437 us
// (5.2 TB/s), with field and gradient 587 us (4.9 TB/s, what the update's own
// 20 streams reach), against 560 and 660 us for a version without the
// following; 64^3, bound by latency, 10.5 against 13.5 us:
// - interior and halo waves in loops of their own; a halo column publishes
//   only the nine values that are gathered from it;
// - the next plane's loads go out as soon as this plane's have been used, the
//   output plane's at the start of the step that completes it, and both have
//   arrived before the step's stores (a wait after them waits for them too);
//   the output plane's a step ahead, before the last stores, measured 1027 us
//   against 912 on 512 x 256 x 256 with walls;
// - an output plane holds its in-plane sums of one slice, then of two (8, then
//   8 and 8 values) in place of three rolling sets of 17;
// - the lattice weights are applied in the gather's sums.
#pragma once
#include "tslb_tiles.h"

namespace tslb {
namespace {

using namespace tile;

// arrival-sensitivity coefficients, order: 1, cx, cy, cz, cx^2, cy^2, cz^2,
// cx cy, cx cz, cy cz
__host__ __device__ inline void arrival_coefficients(const float lam[10], float drho1, const float u[3], float B[10]) {
    const float q = 1.0f / (1.0f + drho1);
    const float ux = u[0], uy = u[1], uz = u[2];
    const float third = 1.0f / 3.0f;
    B[4] = lam[4];
    B[5] = lam[5];
    B[6] = lam[6];
    B[7] = lam[7];
    B[8] = lam[8];
    B[9] = lam[9];
    B[1] = lam[1] * q - 2.0f * lam[4] * ux - lam[7] * uy - lam[8] * uz;
    B[2] = lam[2] * q - 2.0f * lam[5] * uy - lam[7] * ux - lam[9] * uz;
    B[3] = lam[3] * q - 2.0f * lam[6] * uz - lam[8] * ux - lam[9] * uy;
    B[0] = lam[0] - q * (lam[1] * ux + lam[2] * uy + lam[3] * uz) + lam[4] * (ux * ux - third) +
           lam[5] * (uy * uy - third) + lam[6] * (uz * uz - third) + lam[7] * ux * uy + lam[8] * ux * uz +
           lam[9] * uy * uz;
}

// a(c) on the 27 velocities (same separable scheme as the populations: per cz
// slice a quadratic in (cx, cy)); the weights are left to the gather.
__device__ __forceinline__ void arrival_values(const float B[10], float G[27]) {
    eval_slice<0, 27, false>(B[0], B[1], B[2], B[4], B[5], B[7], 0.0f, 0.0f, G);
    const float e0 = B[0] + B[6];
    eval_slice<1, 27, false>(e0 + B[3], B[1] + B[8], B[2] + B[9], B[4], B[5], B[7], 0.0f, 0.0f, G);
    eval_slice<-1, 27, false>(e0 - B[3], B[1] - B[8], B[2] - B[9], B[4], B[5], B[7], 0.0f, 0.0f, G);
}

// The eight in-plane monomial sums of one cz slice F[cy+1][cx+1] of values a,
// sum w F cx^a cy^b, with the lattice weights 216 w = 4^(zero components)
// applied as the factor 4 of every zero component (exact).
struct SliceSums {
    float m00, m10, m01, m20, m02, m11, m21, m12;
    __device__ __forceinline__ void complete() {
        asm volatile("" : "+v"(m00), "+v"(m10), "+v"(m01), "+v"(m20), "+v"(m02), "+v"(m11), "+v"(m21), "+v"(m12));
    }
    // with the slice cz = 0 added
    __device__ __forceinline__ SliceSums plus_middle(const SliceSums& q) const {
        return {fmaf(4.0f, q.m00, m00), fmaf(4.0f, q.m10, m10), fmaf(4.0f, q.m01, m01), fmaf(4.0f, q.m20, m20),
                fmaf(4.0f, q.m02, m02), fmaf(4.0f, q.m11, m11), fmaf(4.0f, q.m21, m21), fmaf(4.0f, q.m12, m12)};
    }
};
__device__ __forceinline__ SliceSums slice_sums(const float F[3][3]) {
    float s[3], d[3], t[3];
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        s[r] = F[r][0] + F[r][2];
        d[r] = F[r][2] - F[r][0];
        t[r] = fmaf(4.0f, F[r][1], s[r]);
    }
    SliceSums q;
    q.m02 = t[2] + t[0];
    q.m00 = fmaf(4.0f, t[1], q.m02);
    q.m01 = t[2] - t[0];
    q.m12 = d[2] + d[0];
    q.m10 = fmaf(4.0f, d[1], q.m12);
    q.m11 = d[2] - d[0];
    q.m20 = fmaf(4.0f, s[1], s[0] + s[2]);
    q.m21 = s[2] - s[0];
    return q;
}

// The 17 weighted monomial moments of the values gathered for one node.
struct AdjSums {
    float L[NK];
    // of the slice cz = -1 (q, the first to reach a node), and the in-plane
    // sums s of it and maybe others with cz = 0
    __device__ __forceinline__ void start(const SliceSums& s, const SliceSums& q) {
        L[K000] = s.m00;
        L[K100] = s.m10;
        L[K010] = s.m01;
        L[K200] = s.m20;
        L[K020] = s.m02;
        L[K110] = s.m11;
        L[K210] = s.m21;
        L[K120] = s.m12;
        L[K001] = -q.m00;
        L[K101] = -q.m10;
        L[K011] = -q.m01;
        L[K201] = -q.m20;
        L[K021] = -q.m02;
        L[K111] = -q.m11;
        L[K002] = q.m00;
        L[K102] = q.m10;
        L[K012] = q.m01;
    }
    template <int CZ>
    __device__ __forceinline__ void add(const SliceSums& q) {
        constexpr float w = CZ == 0 ? 4.0f : 1.0f;
        L[K000] = fmaf(w, q.m00, L[K000]);
        L[K100] = fmaf(w, q.m10, L[K100]);
        L[K010] = fmaf(w, q.m01, L[K010]);
        L[K200] = fmaf(w, q.m20, L[K200]);
        L[K020] = fmaf(w, q.m02, L[K020]);
        L[K110] = fmaf(w, q.m11, L[K110]);
        L[K210] = fmaf(w, q.m21, L[K210]);
        L[K120] = fmaf(w, q.m12, L[K120]);
        if constexpr (CZ != 0) {
            L[K001] += CZ * q.m00;
            L[K101] += CZ * q.m10;
            L[K011] += CZ * q.m01;
            L[K201] += CZ * q.m20;
            L[K021] += CZ * q.m02;
            L[K111] += CZ * q.m11;
            L[K002] += q.m00;
            L[K102] += q.m10;
            L[K012] += q.m01;
        }
    }
};

// The values are complete here: a wait for their loads, or their arithmetic,
// is not moved below this point.
template <int K>
__device__ __forceinline__ void complete(float (&a)[K]) {
#pragma unroll
    for (int k = 0; k < K; ++k) asm volatile("" : "+v"(a[k]));
}

template <bool WALLS, bool FIELD, bool DG, bool NT>
__global__ void __launch_bounds__(NTHREADS, TSLB_WAVES_PER_EU)
    adjoint_tiled_kernel(const float* __restrict__ st0, const float* __restrict__ st1, const float* __restrict__ lam1,
                         float* __restrict__ lam0, float* __restrict__ dg, StepParams p, int tiles_x) {
    static_assert(TX == 64 && 4 + 2 * TY <= 64 && NTHREADS == NINT + 192, "one wave per row, three halo waves");
    __shared__ float lds[NSLOT][LY][LX];
    const Geometry& g = p.geo;
    const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
    const unsigned plane_nodes = (unsigned)nx * (unsigned)ny;
    const size_t stride = (size_t)g.N * 4;
    const bool pz = (g.periodic & 4) != 0;
    // this block's segments (uniform loads); an empty list ends the block
    // before any barrier
    const int4* __restrict__ segs = p.sched + (size_t)blockIdx.x * p.sched_nseg;
    int4 t = segs[0];
    if (t.x < 0) return;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const bool zlo_wall = (g.lo_solid & 4) != 0, zhi_wall = (g.hi_solid & 4) != 0;

    auto solid_col = [&](int wx, int wy) {
        return WALLS && ((wx == 0 && (g.lo_solid & 1)) || (wx == nx - 1 && (g.hi_solid & 1)) ||
                         (wy == 0 && (g.lo_solid & 2)) || (wy == ny - 1 && (g.hi_solid & 2)));
    };
    auto wall_plane = [&](int z) { return WALLS && ((zlo_wall && z == 0) || (zhi_wall && z == nz - 1)); };
    auto plane_of = [&](const float* f, int z) { return f + (size_t)plane_nodes * (size_t)z; };
    auto load_fields = [&]<int K>(const float* f, int z, unsigned node, float (&v)[K]) {
        FieldAddress a(plane_of(f, z), node * 4u);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            v[k] = *a.template lane<const float>();
            a.next(stride);
        }
    };
    // lam and (rho, u) of level t + 1 at a node
    float l[10], u1[4];
    auto fetch = [&](unsigned node, int z) {
        load_fields(lam1, z, node, l);
        load_fields(st1, z, node, u1);
    };
    auto here = [&] {
        __builtin_amdgcn_sched_barrier(0);
        complete(l);
        complete(u1);
        __builtin_amdgcn_sched_barrier(0);
    };
    // Its arrival sensitivities; wall nodes carry none (they never pull
    // populations), con: the column is no wall.
    auto build = [&](float con, int z, float B[10]) {
        if constexpr (WALLS) {
            const float on = wall_plane(z) ? 0.0f : con;
#pragma unroll
            for (int k = 0; k < 10; ++k) l[k] *= on;
        }
        const float u[3] = {u1[1], u1[2], u1[3]};
        arrival_coefficients(l, u1[0], u, B);
    };

    if (wave >= NINT / 64) {
        // ------------------------------------------------------- halo waves
        // One kind of column per wave: the row below the tile (gathered from
        // along cy = -1 only), the row above (cy = +1), then the four corners
        // and the two side columns (cx = -1 on the left, +1 on the right).
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
            float on;
        };
        auto column = [&](int col_id) {
            const int wx = wrap_or_clamp((col_id % tiles_x) * TX - 1 + lx, nx, g.periodic & 1);
            const int wy = wrap_or_clamp((col_id / tiles_x) * TY - 1 + ly, ny, g.periodic & 2);
            return Column{(unsigned)wx + (unsigned)nx * (unsigned)wy, solid_col(wx, wy) ? 0.0f : 1.0f};
        };
        Column c = column(t.x);
        fetch(c.node, plane_index(t.y - 1, nz, pz));
        here();
        float* const w = &lds[0][ly][lx];
        auto put = [&]<int I>(float v) { w[slot_of(I) * LY * LX] = v; };
        for (int k = 0;;) {
            const int4 tn = k + 1 < p.sched_nseg ? segs[k + 1] : make_int4(-1, 0, 0, 0);
            const bool more = tn.x >= 0;
            const Column cn = column(more ? tn.x : t.x);
            const int zs = t.y, ze = t.z;
            for (int zp = zs - 1; zp <= ze; ++zp) {
                float B[10];
                build(c.on, plane_index(zp, nz, pz), B);
                // a(c) with one component fixed at s: a quadratic in the two
                // others, Q[9 + 3 (cz + 1) + (other + 1)]
                float Q[27];
                if (kind != 3) {
                    const float s = kind == 1 ? -1.0f : 1.0f;  // cy
                    eval_slice<0, 27, false>(fmaf(s, B[2], B[0] + B[5]), fmaf(s, B[7], B[1]), fmaf(s, B[9], B[3]), B[4],
                                             B[6], B[8], 0.0f, 0.0f, Q);
                    if (kind == 1)
                        Unroll<0, 27>::run([&]<int I>() {
                            if constexpr (cy_of(I) == -1) put.template operator()<I>(Q[9 + 3 * (cz_of(I) + 1) + cx_of(I) + 1]);
                        });
                    else
                        Unroll<0, 27>::run([&]<int I>() {
                            if constexpr (cy_of(I) == 1) put.template operator()<I>(Q[9 + 3 * (cz_of(I) + 1) + cx_of(I) + 1]);
                        });
                } else {
                    const float s = lx == 0 ? -1.0f : 1.0f;  // cx
                    eval_slice<0, 27, false>(fmaf(s, B[1], B[0] + B[4]), fmaf(s, B[7], B[2]), fmaf(s, B[8], B[3]), B[5],
                                             B[6], B[9], 0.0f, 0.0f, Q);
                    if (publish && lx == 0)
                        Unroll<0, 27>::run([&]<int I>() {
                            if constexpr (cx_of(I) == -1) put.template operator()<I>(Q[9 + 3 * (cz_of(I) + 1) + cy_of(I) + 1]);
                        });
                    if (publish && lx != 0)
                        Unroll<0, 27>::run([&]<int I>() {
                            if constexpr (cx_of(I) == 1) put.template operator()<I>(Q[9 + 3 * (cz_of(I) + 1) + cy_of(I) + 1]);
                        });
                }
                const bool on = zp + 1 <= ze;
                __syncthreads();
                fetch(on ? c.node : cn.node, plane_index(on ? zp + 1 : (more ? tn.y - 1 : ze), nz, pz));
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
        float on;
    };
    auto column = [&](int col_id) {
        Column c;
        c.gx = (col_id % tiles_x) * TX + lane;
        c.gy = (col_id / tiles_x) * TY + wave;
        const int wx = wrap_or_clamp(c.gx, nx, g.periodic & 1);
        const int wy = wrap_or_clamp(c.gy, ny, g.periodic & 2);
        c.node = (unsigned)wx + (unsigned)nx * (unsigned)wy;
        c.on = solid_col(wx, wy) ? 0.0f : 1.0f;
        return c;
    };
    // 1 - omega of plane z: a scalar load (the table is constant here)
    auto omo_of = [&](int z) {
        return p.omo_z ? reinterpret_cast<const __attribute__((address_space(4))) float*>((uintptr_t)p.omo_z)[z]
                       : p.one_minus_omega;
    };
    // moments, acceleration and gradient so far of an output plane
    float m[10], gg[3] = {p.force[0], p.force[1], p.force[2]}, dg_old[3] = {0.0f, 0.0f, 0.0f}, omo = 0.0f;
    auto fetch_out = [&](unsigned node, int z) {
        load_fields(st0, z, node, m);
        if constexpr (FIELD) load_fields(p.gfield, z, node, gg);
        if constexpr (DG) load_fields(dg, z, node, dg_old);
        omo = omo_of(z);
    };

    Column c = column(t.x);
    fetch(c.node, plane_index(t.y - 1, nz, pz));
    here();
    for (int k = 0;;) {
        // the block's next segment: its first plane is loaded during the last
        // plane of this one
        const int4 tn = k + 1 < p.sched_nseg ? segs[k + 1] : make_int4(-1, 0, 0, 0);
        const bool more = tn.x >= 0;
        const Column cn = column(more ? tn.x : t.x);
        const int gx = c.gx, gy = c.gy, zs = t.y, ze = t.z;
        const bool valid = gx < nx && gy < ny;
        const bool col_fluid = valid && !(gy == 0 && ((g.lo_solid | g.lo_ghost) & 2)) &&
                               !(gy == ny - 1 && ((g.hi_solid | g.hi_ghost) & 2)) &&
                               !(gx == 0 && ((g.lo_solid | g.lo_ghost) & 1)) &&
                               !(gx == nx - 1 && ((g.hi_solid | g.hi_ghost) & 1));
        const bool xwalls = WALLS && ((g.lo_solid | g.hi_solid) & 1) != 0;
        const bool ylo = WALLS && (g.lo_solid & 2) && gy == 1, yhi = WALLS && (g.hi_solid & 2) && gy == ny - 2;
        const bool xlo = WALLS && (g.lo_solid & 1) && gx == 1, xhi = WALLS && (g.hi_solid & 1) && gx == nx - 2;

        // Output plane zp - 1 has two of its slices: without walls its
        // in-plane sums (both) and those of its slice cz = -1 (low), with
        // walls, whose terms come from all slices, all of its moments (prev).
        // Output plane zp has its slice cz = -1 (fresh).
        AdjSums prev;
        SliceSums both, low, fresh;
        // Plane zp: publish its arrival sensitivities; what node (col, zp -
        // cz) gathers along (cx, cy, cz) is at (col + (cx, cy), zp), so slice
        // cz of plane zp goes to output plane zp - cz.  PART 1: the halo
        // plane zs - 1, whose slice cz = -1 alone is of use; PART 2: the halo
        // plane ze, its slice cz = +1; PART 3: plane zs, which completes no
        // output plane; 0: the others.
        auto plane = [&]<int PART>(int zp) {
            constexpr auto moves = [](int I) { return PART == 1 ? cz_of(I) == -1 : PART == 2 ? cz_of(I) == 1 : true; };
            const bool on = zp + 1 <= ze;
            const int z1 = plane_index(on ? zp + 1 : (more ? tn.y - 1 : ze), nz, pz);
            float G[27];
            {
                float B[10];
                build(c.on, plane_index(zp, nz, pz), B);
                __builtin_amdgcn_sched_barrier(0);
                fetch(on ? c.node : cn.node, z1);
                if constexpr (PART == 0 || PART == 2) fetch_out(c.node, zp - 1);
                arrival_values(B, G);
            }
            AdjSums cur;
            if constexpr (WALLS && (PART == 0 || PART == 3)) cur.start(fresh, fresh);
            if constexpr (WALLS && (PART == 0 || PART == 3)) {
                // own population bounced back: a_y(c_j) arrives as if along
                // -c_j, at fluid nodes only (ghost nodes are never updated)
                const bool zlo = zlo_wall && zp == 1, zhi = zhi_wall && zp == nz - 2;
                const bool plane_fluid = !(zp == 0 && ((g.lo_solid | g.lo_ghost) & 4)) &&
                                         !(zp == nz - 1 && ((g.hi_solid | g.hi_ghost) & 4));
                if ((ylo || yhi || zlo || zhi || xwalls) && plane_fluid && col_fluid) {
                    auto bounce = [&]<int CZ>() {
                        float F[3][3];
                        Unroll<0, 9>::run([&]<int K>() {
                            constexpr int I = 9 * (CZ + 1) + K, J = 26 - I;  // J = -c_I
                            bool s = false;
                            if (cx_of(J) == 1) s |= xlo;
                            if (cx_of(J) == -1) s |= xhi;
                            if (cy_of(J) == 1) s |= ylo;
                            if (cy_of(J) == -1) s |= yhi;
                            if (cz_of(J) == 1) s |= zlo;
                            if (cz_of(J) == -1) s |= zhi;
                            F[cy_of(I) + 1][cx_of(I) + 1] = s ? G[J] : 0.0f;
                        });
                        cur.template add<CZ>(slice_sums(F));
                    };
                    bounce.template operator()<-1>();
                    bounce.template operator()<0>();
                    bounce.template operator()<1>();
                }
            }
            Unroll<0, 27>::run([&]<int I>() {
                if constexpr ((cx_of(I) != 0 || cy_of(I) != 0) && moves(I)) lds[slot_of(I)][ly][lx] = G[I];
            });
            __syncthreads();
            // the arriving values go to registers at once, so the buffer is
            // free again after the second barrier
            float F[3][3][3];  // [cz + 1][cy + 1][cx + 1]
            Unroll<0, 27>::run([&]<int I>() {
                constexpr int X = cx_of(I), Y = cy_of(I), Z = cz_of(I);
                if constexpr (!moves(I))
                    F[Z + 1][Y + 1][X + 1] = 0.0f;
                else if constexpr (X == 0 && Y == 0)
                    F[Z + 1][1][1] = G[I];
                else
                    F[Z + 1][Y + 1][X + 1] = lds[slot_of(I)][ly + Y][lx + X];
            });
            __syncthreads();
            __builtin_amdgcn_sched_barrier(0);
            AdjSums done;
            if constexpr (PART == 0 || PART == 2) {
                if constexpr (WALLS)
                    done = prev;
                else
                    done.start(both, low);
                done.template add<1>(slice_sums(F[2]));
            }
            if constexpr (PART == 0 || PART == 3) {
                if constexpr (WALLS) {
                    cur.template add<0>(slice_sums(F[1]));
                    prev = cur;
                    complete(prev.L);
                } else {
                    both = fresh.plus_middle(slice_sums(F[1]));
                    low = fresh;
                    both.complete();
                }
            }
            if constexpr (PART != 2) {
                fresh = slice_sums(F[0]);
                fresh.complete();
            }
            if constexpr (PART == 0 || PART == 2) {
                const int zo = zp - 1;
                float out[10], lg[3];
#pragma unroll
                for (int k = 0; k < NK; ++k) done.L[k] *= kInv216;
                coefficients_vjp(done.L, m, gg, omo, out, lg);
                float dgn[3];
#pragma unroll
                for (int a = 0; a < 3; ++a) dgn[a] = dg_old[a] + lg[a];
                // every node that emits (fluid or ghost) has a sensitivity;
                // walls emit nothing
                const bool emits = !WALLS || (c.on != 0.0f && !wall_plane(zo));
                complete(out);
                if constexpr (DG) complete(dgn);
                __builtin_amdgcn_sched_barrier(0);
                // before the stores: a wait after them would wait for those too
                here();
                if (valid) {
                    FieldAddress o(plane_of(lam0, zo), c.node * 4u);
#pragma unroll
                    for (int q = 0; q < 10; ++q) {
                        store_out<NT>(o.template lane<float>(), emits ? out[q] : 0.0f);
                        o.next(stride);
                    }
                    if constexpr (DG) {
                        if (emits) {
                            FieldAddress d(plane_of(dg, zo), c.node * 4u);
#pragma unroll
                            for (int a = 0; a < 3; ++a) {
                                store_out<NT>(d.template lane<float>(), dgn[a]);
                                d.next(stride);
                            }
                        }
                    }
                }
            }
        };
        plane.template operator()<1>(zs - 1);
        plane.template operator()<3>(zs);
        for (int zp = zs + 1; zp < ze; ++zp) plane.template operator()<0>(zp);
        plane.template operator()<2>(ze);
        if (!more) return;
        ++k;
        t = tn;
        c = cn;
    }
}

template <bool WALLS, bool FIELD, bool DG>
hipError_t launch_t(const float* st0, const float* st1, const float* lam1, float* lam0, float* dg,
                    const StepParams& p, hipStream_t s) {
    if (p.geo.N >= (1LL << 30)) return hipErrorInvalidValue;  // 32-bit byte offsets
    if (!p.sched || p.sched_grid < 8 || p.sched_nseg < 1) return hipErrorInvalidValue;
    const int tiles_x = (p.geo.n[0] + TX - 1) / TX;
    if (((long long)p.geo.n[0] * 4) % 128 == 0)
        hipLaunchKernelGGL((adjoint_tiled_kernel<WALLS, FIELD, DG, true>), dim3(p.sched_grid), dim3(NTHREADS), 0, s,
                           st0, st1, lam1, lam0, dg, p, tiles_x);
    else
        hipLaunchKernelGGL((adjoint_tiled_kernel<WALLS, FIELD, DG, false>), dim3(p.sched_grid), dim3(NTHREADS), 0, s,
                           st0, st1, lam1, lam0, dg, p, tiles_x);
    return hipGetLastError();
}

template <bool WALLS>
hipError_t launch_w(const float* st0, const float* st1, const float* lam1, float* lam0, float* dg,
                    const StepParams& p, hipStream_t s) {
    const bool field = p.gfield != nullptr;
    if (dg)
        return field ? launch_t<WALLS, true, true>(st0, st1, lam1, lam0, dg, p, s)
                     : launch_t<WALLS, false, true>(st0, st1, lam1, lam0, dg, p, s);
    return field ? launch_t<WALLS, true, false>(st0, st1, lam1, lam0, dg, p, s)
                 : launch_t<WALLS, false, false>(st0, st1, lam1, lam0, dg, p, s);
}

hipError_t launch_adjoint(const float* st0, const float* st1, const float* lam1, float* lam0, float* dg,
                          const StepParams& p, hipStream_t s) {
    if ((p.geo.lo_solid | p.geo.hi_solid) != 0) return launch_w<true>(st0, st1, lam1, lam0, dg, p, s);
    return launch_w<false>(st0, st1, lam1, lam0, dg, p, s);
}

}  // namespace
}  // namespace tslb
