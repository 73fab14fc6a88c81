// D2Q9 form of the moment-only thread-safe update (the two-dimensional
// counterpart of D3Q27 that Section 2.2 names): the tensor product of the
// three-point weights in x and y, the same Hermite reconstruction (up to
// third order; H_xxx vanishes on this lattice as on D3Q27) and the same
// BGK relaxation and forcing.  The state keeps the 10-field layout with
// nz = 1; the update reads and writes the six fields drho, u_x, u_y,
// Pi_xx, Pi_yy, Pi_xy only (u_z and the Pi components with a z index stay
// zero).
//
// Kernel shape: one wavefront owns a span of 64 or 128 x-columns (one or two
// per lane, 64 apart, so that every load is whole cache lines) and marches a
// segment of rows along y.  For every row it builds the 9 populations of its
// nodes (without their weights, which the sums apply), moves the ones with
// c_x != 0 to their x-neighbour across lanes (no LDS, no block barrier; the
// two edge lanes rebuild the three values that enter from the neighbouring
// spans), and adds each c_y slice to the row it arrives in (rows y - 1, y,
// y + 1).  Row y - 1 is then complete and is finalised and stored.  Walls:
// wall nodes are stored as the rest state and emit nothing; a fluid node next
// to a wall adds its own bounced-back populations, straight from the nine it
// has just built, to its own row (half-way bounce-back).
//
// What bounds it (8192 x 4096 channel): memory with FP32 storage, 320 us (5.0
// TB/s), arithmetic with FP16, 194 us.  It took 351 and 225 us with one
// column per lane (the edge lanes' node costs the wave as much as its own),
// nine values summed one by one, shifts through LDS permutes, a second load
// round trip for the edge lanes and stores ahead of the next row's loads (a
// wait for loads waits for the stores before them): now the next row's loads
// go out once this row's have been used and have arrived before its stores.
#include <algorithm>

#include "tslb_internal.h"

namespace tslb {
namespace {

constexpr int kD2Block = 256;          // four independent wavefronts


// One c_y slice of arriving deviations (c_x = -1, 0, 1), without lattice
// weights, reduced along x: sum, sum c_x and sum c_x^2 with the factor 4 of a
// zero component applied (36 w = 4^n0).
struct Slice2 {
    float t, d, s;
};
__device__ __forceinline__ Slice2 slice2(float m, float z, float p) {
    const float s = p + m;
    return {fmaf(4.0f, z, s), p - m, s};
}

// Moment sums of the arriving scaled deviations (2D).
struct Sums2 {
    float d, jx, jy, sxx, syy, sxy;
    // the slices c_y = +1 (q, the first to reach a row), 0 and -1
    __device__ __forceinline__ void start(const Slice2& q) {
        d = jy = syy = q.t;
        jx = sxy = q.d;
        sxx = q.s;
    }
    __device__ __forceinline__ void middle(const Slice2& q) {
        d = fmaf(4.0f, q.t, d);
        jx = fmaf(4.0f, q.d, jx);
        sxx = fmaf(4.0f, q.s, sxx);
    }
    __device__ __forceinline__ void finish(const Slice2& q) {
        d += q.t;
        jx += q.d;
        jy -= q.t;
        sxx += q.s;
        syy += q.t;
        sxy -= q.d;
    }
    // one arriving value, weight applied
    template <int CX, int CY>
    __device__ __forceinline__ void add(float f) {
        d += f;
        if (CX) {
            jx += CX * f;
            sxx += f;
        }
        if (CY) {
            jy += CY * f;
            syy += f;
        }
        if (CX * CY) sxy += CX * CY * f;
    }
    __device__ __forceinline__ void complete() {
        asm volatile("" : "+v"(d), "+v"(jx), "+v"(jy), "+v"(sxx), "+v"(syy), "+v"(sxy));
    }
};

// Population polynomial of one node, G(c) = 36 w(c) P(c): P is the
// polynomial of the D3Q27 kernels with every z component zero (the
// expression does not depend on the dimension),
//   P = b00 + b10 cx + b01 cy + b20 cx^2 + b02 cy^2 + b11 cx cy
//       + b21 cx^2 cy + b12 cx cy^2,
// from the equilibrium rho [3 cu + 9/2 cu^2 - 3/2 u^2 + 9/2 cu^3 - 9/2 cu u^2]
// and the non-equilibrium part (1 - omega) [9/2 cPc - 3/2 tr Pi +
// 27/2 cPc cu - 9/2 tr Pi cu - 9 c.Pi u] with c_a^3 = c_a, plus 3 rho c.g.
// ORDER 2 keeps the terms up to H2 (the cubic monomials vanish and the
// linear ones reduce to 3 rho (u + g)).  m = (drho, u_x, u_y, Pi_xx, Pi_yy,
// Pi_xy); b = (b00, b10, b01, b20, b02, b11, b21, b12).
template <int ORDER>
__device__ __forceinline__ void coefficients2(const float m[6], float gx, float gy, float omo, float b[8]) {
    const float dr = m[0], rho = 1.0f + dr, ux = m[1], uy = m[2];
    const float pxx = omo * m[3], pyy = omo * m[4], pxy = omo * m[5];
    const float rx = rho * ux, ry = rho * uy;
    const float u2 = ux * ux + uy * uy, tr = pxx + pyy;
    b[0] = dr - 1.5f * (rho * u2 + tr);
    b[3] = 4.5f * (rx * ux + pxx);
    b[4] = 4.5f * (ry * uy + pyy);
    b[5] = 9.0f * (rx * uy + pxy);
    if constexpr (ORDER < 3) {
        b[1] = 3.0f * (rx + rho * gx);
        b[2] = 3.0f * (ry + rho * gy);
        b[6] = b[7] = 0.0f;
        return;
    }
    // 27/2 (rho u_a^2 u_b + Pi_aa u_b + 2 Pi_ab u_a) = 3 b_aa u_b + 27 Pi_ab u_a;
    // the Pi_aa u_a terms of the linear coefficients collapse into b_aa u_a
    const float base = 3.0f - 4.5f * u2, t45 = 4.5f * tr, qxy = 27.0f * pxy;
    b[1] = rx * base + ux * (b[3] - t45) - 9.0f * pxy * uy + 3.0f * rho * gx;
    b[2] = ry * base + uy * (b[4] - t45) - 9.0f * pxy * ux + 3.0f * rho * gy;
    b[6] = 3.0f * b[3] * uy + qxy * ux;
    b[7] = 3.0f * b[4] * ux + qxy * uy;
}

// G[3 (cy + 1) + (cx + 1)] = P(cx, cy), without the weight: along x for each
// power of cy, then along y.
__device__ __forceinline__ void populations2(const float b[8], float G[9]) {
    const float s0 = b[0] + b[3], s1 = b[2] + b[6];
    const float r0[3] = {s0 - b[1], b[0], s0 + b[1]};
    const float r1[3] = {s1 - b[5], b[2], s1 + b[5]};
    const float r2[3] = {b[4] - b[7], b[4], b[4] + b[7]};
#pragma unroll
    for (int ix = 0; ix < 3; ++ix) {
        const float t = r0[ix] + r2[ix];
        const float q[3] = {t - r1[ix], r0[ix], t + r1[ix]};
#pragma unroll
        for (int iy = 0; iy < 3; ++iy) G[3 * iy + ix] = q[iy];
    }
}

// v of the next lane (wave_shr:1 0x138: the lane on the left, wave_shl:1
// 0x130: on the right); the end lane without one gets h.
template <int CTRL>
__device__ __forceinline__ float shift_lane(float v, float h) {
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(h), __float_as_int(v), CTRL, 0xf, 0xf, false));
}

// v of one lane, in all of them.
__device__ __forceinline__ float lane_value(float v, int lane) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

// Per-field base pointers of the six stored D2Q9 fields (drho, u_x, u_y,
// Pi_xx, Pi_yy, Pi_xy: fields 0, 1, 2, 4, 5, 7 of the ten-field state) and
// of the force field, passed as a kernel argument so every base sits in
// scalar registers and each access is that base plus one 32-bit byte offset.
template <class T>
struct Fields2 {
    const T* in[6];
    T* out[6];
    const float* g[2];
};

// One node's stored values as they come from memory, and its force.
template <class T>
struct Raw2 {
    T m[6];
    float g[2];
};

template <bool FIELD, class T>
__device__ __forceinline__ void fetch2(const Fields2<T>& f, unsigned off, Raw2<T>& r) {
#pragma unroll
    for (int k = 0; k < 6; ++k) r.m[k] = *(const T*)((const char*)f.in[k] + off);
    if constexpr (FIELD) {
        r.g[0] = *(const float*)((const char*)f.g[0] + (off / sizeof(T)) * 4u);
        r.g[1] = *(const float*)((const char*)f.g[1] + (off / sizeof(T)) * 4u);
    }
}

template <class S>
__device__ __forceinline__ void decode2(const Raw2<typename S::T>& r, const StepParams& p, float m[6]) {
    m[0] = S::load(r.m[0], p.inv_scale[0]);
#pragma unroll
    for (int k = 1; k < 3; ++k) m[k] = S::load(r.m[k], p.inv_scale[1]);
#pragma unroll
    for (int k = 3; k < 6; ++k) m[k] = S::load(r.m[k], p.inv_scale[2]);
}

// The loaded values are needed from here on: the wait for them stands here,
// ahead of the stores that follow.
template <bool FIELD, class T>
__device__ __forceinline__ void arrive2(Raw2<T>& r) {
#pragma unroll
    for (int k = 0; k < 6; ++k) asm volatile("" : "+v"(r.m[k]));
    if constexpr (FIELD) asm volatile("" : "+v"(r.g[0]), "+v"(r.g[1]));
}

__device__ __forceinline__ int wrap_clamp(int v, int n, bool periodic) {
    if (periodic) {
        v %= n;
        return v < 0 ? v + n : v;
    }
    return v < 0 ? 0 : (v >= n ? n - 1 : v);
}

// Output stores, non-temporal or plain (see launch_o).
template <bool NT, class T>
__device__ __forceinline__ void out_store(T* p, T v) {
    if constexpr (!NT)
        *p = v;
    else if constexpr (sizeof(T) == 4)
        __builtin_nontemporal_store(__builtin_bit_cast(float, v), reinterpret_cast<float*>(p));
    else
        __builtin_nontemporal_store(__builtin_bit_cast(unsigned short, v), reinterpret_cast<unsigned short*>(p));
}

template <class S, int ORDER, bool FIELD, bool NT, int C>
__global__ void __launch_bounds__(kD2Block) update_d2q9_kernel(const Fields2<typename S::T> f, StepParams p, int spans,
                                                               int segments, int seg_rows) {
    using T = typename S::T;
    const Geometry& g = p.geo;
    const int nx = g.n[0], ny = g.n[1];
    const int lane = threadIdx.x & 63;
    // Block ids are dealt round-robin to the 8 XCDs (the grid is a multiple
    // of 8 blocks); each XCD takes a contiguous run of blocks, so the spans
    // that march side by side share an L2 and the halo columns the edge
    // lanes read are mostly hits.
    const int per = (int)(gridDim.x >> 3);
    const int vb = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
    const int item = vb * (kD2Block / 64) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (item >= spans * segments) return;  // whole wavefronts leave together
    const int span = item % spans, seg = item / spans;
    const int y0 = seg * seg_rows, y1 = min(y0 + seg_rows, ny);
    const int x0 = span * (64 * C);
    const bool px = (g.periodic & 1) != 0, py = (g.periodic & 2) != 0;
    // The edge lanes also rebuild the populations that enter the span from
    // the neighbouring columns: lane 0 those with c_x = +1 of node x0 - 1,
    // lane 63 those with c_x = -1 of node x0 + 64 C.
    const bool edge = lane == 0 || lane == 63;
    const int hx = wrap_clamp(lane == 0 ? x0 - 1 : x0 + 64 * C, nx, px);
    const float hs = lane == 0 ? 1.0f : -1.0f;
    auto solid_at = [&](int x) { return (x == 0 && (g.lo_solid & 1)) || (x == nx - 1 && (g.hi_solid & 1)); };
    const bool hsolid_col = solid_at(hx);
    int x[C];  // lanes past the last column build the node the periodic wrap or the
               // clamp puts there (its populations still reach the last column)
    bool col_solid[C], fluid_col[C], wl[C], wr[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const int gx = x0 + 64 * c + lane;
        x[c] = wrap_clamp(gx, nx, px);
        col_solid[c] = solid_at(x[c]);
        fluid_col[c] = gx < nx && !col_solid[c] && !(x[c] == 0 && (g.lo_ghost & 1)) && !(x[c] == nx - 1 && (g.hi_ghost & 1));
        wl[c] = (g.lo_solid & 1) && x[c] == 1;
        wr[c] = (g.hi_solid & 1) && x[c] == nx - 2;
    }
    const float omo = omo_at(p, 0);

    Raw2<T> own[C], side;  // row yp on entry to row(yp); side: the edge lanes' neighbour
#pragma unroll
    for (int k = 0; k < 6; ++k) side.m[k] = T{};
    side.g[0] = side.g[1] = 0.0f;
    auto fetch = [&](int yp) {
        const unsigned r = (unsigned)(nx * wrap_clamp(yp, ny, py));  // byte offsets < 2^32: N < 2^30
        if (edge) fetch2<FIELD>(f, ((unsigned)hx + r) * (unsigned)sizeof(T), side);
#pragma unroll
        for (int c = 0; c < C; ++c) fetch2<FIELD>(f, ((unsigned)x[c] + r) * (unsigned)sizeof(T), own[c]);
    };
    // prev: row yp - 1 with two of its slices; fresh: the slice c_y = +1 of row yp
    Sums2 prev[C];
    Slice2 fresh[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
        fresh[c] = {0.0f, 0.0f, 0.0f};
        prev[c].start(fresh[c]);
    }
    fetch(y0 - 1);
    for (int yp = y0 - 1; yp <= y1; ++yp) {
        const int y = wrap_clamp(yp, ny, py);
        const bool row_solid = (y == 0 && (g.lo_solid & 2)) || (y == ny - 1 && (g.hi_solid & 2));
        auto build = [&](const Raw2<T>& r, bool solid, float b[8]) {
            float m[6];
            decode2<S>(r, p, m);
            const float gx = solid ? 0.0f : FIELD ? r.g[0] : p.force[0];
            const float gy = solid ? 0.0f : FIELD ? r.g[1] : p.force[1];
            coefficients2<ORDER>(m, gx, gy, omo, b);
        };
        // halo values H[cy + 1] = P(hs, cy) of node (hx, y), with
        // P(s, cy) = r0 + cy r1 + cy^2 r2
        float H[3] = {0.0f, 0.0f, 0.0f};
        if (edge) {
            float b[8];
            build(side, hsolid_col || row_solid, b);
            const float r0 = b[0] + hs * b[1] + b[3], r1 = b[2] + hs * b[5] + b[6], r2 = b[4] + hs * b[7];
            const float t2 = r0 + r2;
            H[0] = t2 - r1;
            H[1] = r0;
            H[2] = t2 + r1;
        }
        float G[C][9];
#pragma unroll
        for (int c = 0; c < C; ++c) {
            float b[8];
            build(own[c], col_solid[c] || row_solid, b);
            populations2(b, G[c]);
        }
        __builtin_amdgcn_sched_barrier(0);
        fetch(min(yp + 1, y1));  // past the last row: that row again, not used
        const int yo = yp - 1;   // the row this one completes
        const bool out_row = yo >= y0 && !(yo == 0 && ((g.lo_solid | g.lo_ghost) & 2)) &&
                             !(yo == ny - 1 && ((g.hi_solid | g.hi_ghost) & 2));
        T o[C][6];
#pragma unroll
        for (int c = 0; c < C; ++c) {
            // arrivals of slice cy: c_x = +1 from the lane on the left, -1
            // from the lane on the right, across the column sets through the
            // lane at their border
            auto arrive = [&]<int CY>() {
                constexpr int r = 3 * (CY + 1);
                const float hl = c == 0 ? H[CY + 1] : lane_value(G[c == 0 ? 0 : c - 1][r + 2], 63);
                const float hr = c == C - 1 ? H[CY + 1] : lane_value(G[c == C - 1 ? c : c + 1][r], 0);
                return slice2(shift_lane<0x130>(G[c][r], hr), G[c][r + 1], shift_lane<0x138>(G[c][r + 2], hl));
            };
            Sums2 a = prev[c];
            a.finish(arrive.template operator()<-1>());  // row yp - 1
            Sums2& cur = prev[c];
            cur.start(fresh[c]);
            cur.middle(arrive.template operator()<0>());  // row yp
            fresh[c] = arrive.template operator()<1>();   // row yp + 1
            // half-way bounce-back: a fluid node next to a wall receives its
            // own population along -c for every c whose upstream node x - c
            // is a wall; it arrives in the node's own row
            const bool wb = (g.lo_solid & 2) && yp == 1, wt = (g.hi_solid & 2) && yp == ny - 2;
            if (fluid_col[c] && !row_solid && (wl[c] || wr[c] || wb || wt)) {
#define TSLB_BB(I, X, Y)                                                                  \
    if ((X == 1 && wl[c]) || (X == -1 && wr[c]) || (Y == 1 && wb) || (Y == -1 && wt)) \
        cur.template add<X, Y>(((X == 0) + (Y == 0) == 1 ? 4.0f : 1.0f) * G[c][8 - I]);
                TSLB_BB(0, -1, -1)
                TSLB_BB(1, 0, -1)
                TSLB_BB(2, 1, -1)
                TSLB_BB(3, -1, 0)
                TSLB_BB(5, 1, 0)
                TSLB_BB(6, -1, 1)
                TSLB_BB(7, 0, 1)
                TSLB_BB(8, 1, 1)
#undef TSLB_BB
            }
            cur.complete();
            // drho' = D/36, u' = J/(36 + D), Pi' = (S - J u' - D/3 delta)/36
            const float den = 36.0f + a.d;
            float inv = __builtin_amdgcn_rcpf(den);
            inv = inv * fmaf(-den, inv, 2.0f);
            const float ux = a.jx * inv, uy = a.jy * inv, d3 = a.d * (1.0f / 3.0f);
            constexpr float k36 = 1.0f / 36.0f;
            o[c][0] = S::store(a.d * k36, p.scale[0]);
            o[c][1] = S::store(ux, p.scale[1]);
            o[c][2] = S::store(uy, p.scale[1]);
            o[c][3] = S::store((a.sxx - a.jx * ux - d3) * k36, p.scale[2]);
            o[c][4] = S::store((a.syy - a.jy * uy - d3) * k36, p.scale[2]);
            o[c][5] = S::store((a.sxy - a.jx * uy) * k36, p.scale[2]);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < C; ++c) arrive2<FIELD>(own[c]);
        arrive2<FIELD>(side);
        __builtin_amdgcn_sched_barrier(0);
        if (!out_row) continue;
#pragma unroll
        for (int c = 0; c < C; ++c) {
            if (!fluid_col[c]) continue;
            const unsigned oo = (unsigned)(x[c] + nx * yo) * (unsigned)sizeof(T);
#pragma unroll
            for (int k = 0; k < 6; ++k) out_store<NT>((T*)((char*)f.out[k] + oo), o[c][k]);
        }
    }
}

// Spans and segments.  The chip takes 4096 wavefronts at 16 per CU; rows per
// segment so that there are as many, down to one row: at least three rows of
// loads in a chain (256 x 256: 5.2 us; with segments of 16 rows 18.6).  Up to
// four rows in all are not cut where the spans alone give each CU four
// wavefronts: a cut costs two rows of halo (100000 x 3: 8.3 us, 11.4 cut).
// Two columns per lane where that still leaves segments of eight rows (8192 x
// 4096: 320 us, 343 with one column; 512 x 512 7.0 and 6.8) or, of up to four
// rows, 4096 wavefronts (2^22 x 2: 100 and 110), and at most a ninth of the
// columns more (3 x 100000: 38 us with one column, 64 with two;
// 64 x 65536 36 and 49).  FP32, bound by memory, takes up to 32 rows at eight
// wavefronts per CU instead, for fewer halo rows (4096 x 2048: 82.4 us with 32
// rows, 85.2 with 16), but no number between (128 x 100000: 133 us with 25
// rows, 162 with 32, which give three blocks to some CUs and four to others);
// 16-bit storage, bound by arithmetic, does not (2048 x 2048 FP16: 28.6 us
// with 8 rows, 33.0 with 16).
template <class S, int ORDER, bool FIELD, bool NT>
hipError_t launch_c(const Fields2<typename S::T>& f, const StepParams& p, hipStream_t s) {
    const int nx = p.geo.n[0], ny = p.geo.n[1];
    constexpr long long kWaves = 4096;
    auto rows = [&](int spans) {
        return ny <= 4 && spans >= kWaves / 4 ? ny : (int)std::max(1LL, ((long long)ny * spans + kWaves - 1) / kWaves);
    };
    auto run = [&]<int C>(int seg_rows) {
        const int spans = (nx + 64 * C - 1) / (64 * C), segments = (ny + seg_rows - 1) / seg_rows;
        const long long waves = (long long)spans * segments;
        const unsigned blocks = (unsigned)((waves + kD2Block / 64 - 1) / (kD2Block / 64));
        const unsigned grid = (blocks + 7u) & ~7u;  // a multiple of 8: whole runs per XCD
        hipLaunchKernelGGL((update_d2q9_kernel<S, ORDER, FIELD, NT, C>), dim3(grid), dim3(kD2Block), 0, s, f, p, spans,
                           segments, seg_rows);
        return hipGetLastError();
    };
    const int one = (nx + 63) / 64, two = (nx + 127) / 128, r2 = rows(two);
    const bool full = r2 >= 8 || (ny <= 4 && two >= kWaves);
    if (!full || 9 * (2 * two - one) > one) return run.template operator()<1>(rows(one));
    return run.template operator()<2>(sizeof(typename S::T) == 4 && r2 <= 16 ? 2 * r2 : r2);
}

template <class S, int ORDER>
hipError_t launch_o(const void* in, void* out, const StepParams& p, hipStream_t s) {
    using T = typename S::T;
    const size_t N = (size_t)p.geo.N;
    Fields2<T> f;
    const int field[6] = {0, 1, 2, 4, 5, 7};
    for (int k = 0; k < 6; ++k) {
        f.in[k] = (const T*)in + field[k] * N;
        f.out[k] = (T*)out + field[k] * N;
    }
    for (int a = 0; a < 2; ++a) f.g[a] = p.gfield ? p.gfield + a * N : nullptr;
    // Non-temporal stores (the new level is not read again by this launch)
    // when every row is whole cache lines, so that no line is completed by a
    // neighbour, and the two levels do not fit the Infinity Cache, where the
    // next step finds them (2048 x 2048, 201 MB: 47.0 us non-temporal, 35.1
    // plain; 16384 x 1024, 805 MB: 157 and 162).
    const bool nt = (p.geo.n[0] * sizeof(T)) % 128 == 0 && 12 * N * sizeof(T) > kInfinityCacheBytes;
    if (p.gfield) return nt ? launch_c<S, ORDER, true, true>(f, p, s) : launch_c<S, ORDER, true, false>(f, p, s);
    return nt ? launch_c<S, ORDER, false, true>(f, p, s) : launch_c<S, ORDER, false, false>(f, p, s);
}

template <class S>
hipError_t launch_s(const void* in, void* out, const StepParams& p, hipStream_t s) {
    return p.order == 2 ? launch_o<S, 2>(in, out, p, s) : launch_o<S, 3>(in, out, p, s);
}

}  // namespace

hipError_t launch_update_d2q9(int storage, const void* in, void* out, const StepParams& p, hipStream_t s) {
    if (p.geo.n[2] != 1 || p.geo.N >= (1LL << 30)) return hipErrorInvalidValue;  // 32-bit byte offsets
    switch (storage) {
    case 0: return launch_s<StoreF32>(in, out, p, s);
    case 1: return launch_s<StoreF16>(in, out, p, s);
    case 2: return launch_s<StoreBF16>(in, out, p, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace tslb
