// (2+1)D: several time steps per pass on one tile held in registers (Sect. 3,
// Eqs. scheme2Deq-scheme4thline), shared by the single-lattice kernel and the
// batched kernels.
//
// A workgroup of NW waves covers a region of 64 x (NW K) cells: the tile plus a
// ring of `ring` cells on each side.  Lane l of wave w owns column l of rows
// w K .. w K + K - 1 for the whole pass: its amplitudes and coefficients are
// loaded once, stay in registers for all steps and the tile's are stored once.
// A half-step needs one x and one y neighbour of each array: x neighbours come
// from the next lane (a DPP wave shift, no LDS), y neighbours inside the
// thread's rows from its own registers, and only the first and last row of each
// wave go through LDS (double-buffered, one barrier per half-step).
//
// Every half-step is evaluated on the whole region.  The cells at its rim use
// neighbours that are not there, and a wrong value moves one cell inwards per
// full step (each half-step reaches one cell in one direction per axis, and the
// two half-steps reach in opposite ones), so after `steps` <= ring steps the
// tile is untouched by it.  Region cells outside the lattice hold the periodic
// images (loaded wrapped, then advanced like any other cell, also where the
// region is larger than the lattice) or, with zero values outside, stay zero.
//
// What bounds it: on small lattices the launch (about 3 us) and the latency of a
// half-step (0.35 us with 16 rows per workgroup).  On large ones neither the vector ALUs
// nor the bus alone: a workgroup loads, steps and stores one after the other, and two on
// a CU hide little of that.  By the counters a pass of 1024 x 512 complex64 per site issues
// vector instructions for 9.2 of its 18 us, of 2047 x 1531 for 51 of 80 (its bytes take 53),
// of 15 lattices of 6.4 M cells together for 130 of 180.  A region cell takes 77
// instructions a step (complex64 per site), 72 of them the update, shifts between lanes
// being folded into it; with the rim that is 142 per cell of the lattice.  Per step,
// measured next to the row marches (one or two steps per pass) on one box:
//   128 x 128 complex128, no potential     1.17 us (7 steps per pass)  5.2 us
//   512 x 512 complex64, per site          2.15 us (5)                 9.6 us
//   1024 x 512 complex64, per site         3.50 us (5)                10.3 us
//   2047 x 1531 complex64, per site        14.1 us (6)                68.7 us
//   2048 x 2048 complex128, per site       45.9 us (6)                79.8 us
//   4096 x 4096 complex64, per site        72.7 us (6)               173.5 us
// Three shapes (K, NW) are built: (1, 16) spreads a small lattice over most
// workgroups and lets whole waves skip rows that no longer matter, (6, 8) wastes
// least on the ring of a large one, (2, 16) between them and where (6, 8) would
// not fit the registers (complex128 per site).  (4, 8), (5, 8) and (8, 8) came
// out within 5% of one of the three at every size, never ahead by more.
//
// The helpers and the operation order are those of the one-step kernels, so the
// result is bitwise that of the same number of one-step passes, forward and
// reversed (v then u, with r, theta negated).
#pragma once

#include "device.h"
#include "internal.h"
#include "march2.h"
#include "ntstore.h"
#include "stencil3.h"

namespace dirac {

// Value of the lane below (i - 1) or above (i + 1); the rim lanes get zero.
__device__ __forceinline__ int t2_from_below(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x138, 0xf, 0xf, true); }
__device__ __forceinline__ int t2_from_above(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x130, 0xf, 0xf, true); }
__device__ __forceinline__ float t2_xm(float v) { return __int_as_float(t2_from_below(__float_as_int(v))); }
__device__ __forceinline__ float t2_xp(float v) { return __int_as_float(t2_from_above(__float_as_int(v))); }
__device__ __forceinline__ double t2_xm(double v) {
    return __hiloint2double(t2_from_below(__double2hiint(v)), t2_from_below(__double2loint(v)));
}
__device__ __forceinline__ double t2_xp(double v) {
    return __hiloint2double(t2_from_above(__double2hiint(v)), t2_from_above(__double2loint(v)));
}
template <typename C> __device__ __forceinline__ C t2_cxm(C v) { return mk2(t2_xm(v.x), t2_xm(v.y)); }
template <typename C> __device__ __forceinline__ C t2_cxp(C v) { return mk2(t2_xp(v.x), t2_xp(v.y)); }

// The same around the wave: the first lane's lower neighbour is the last lane.
__device__ __forceinline__ int t2_rot_below(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x13c, 0xf, 0xf, true); }
__device__ __forceinline__ int t2_rot_above(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x134, 0xf, 0xf, true); }
__device__ __forceinline__ float t2_rm(float v) { return __int_as_float(t2_rot_below(__float_as_int(v))); }
__device__ __forceinline__ float t2_rp(float v) { return __int_as_float(t2_rot_above(__float_as_int(v))); }
__device__ __forceinline__ double t2_rm(double v) {
    return __hiloint2double(t2_rot_below(__double2hiint(v)), t2_rot_below(__double2loint(v)));
}
__device__ __forceinline__ double t2_rp(double v) {
    return __hiloint2double(t2_rot_above(__double2hiint(v)), t2_rot_above(__double2loint(v)));
}
template <typename C> __device__ __forceinline__ C t2_rxm(C v) { return mk2(t2_rm(v.x), t2_rm(v.y)); }
template <typename C> __device__ __forceinline__ C t2_rxp(C v) { return mk2(t2_rp(v.x), t2_rp(v.y)); }

// The Cayley coefficients of coef_theta(th), bit for bit, with the reciprocal of
// 1 + th^2 written out: the hardware's estimate, two Newton steps and the residual
// correction, which are the steps of an IEEE division whose operands need no
// scaling (1 + th^2 is at least 1; the scaling, its undoing and the fix-up of
// special operands are quarter-rate instructions).
__device__ __forceinline__ Coef<double> coef_theta_r(double th) {
    const double t2 = th * th, d = 1.0 + t2;
    double y = __builtin_amdgcn_rcp(d);
    y = fmx(y, fmx(-d, y, 1.0), y);
    y = fmx(y, fmx(-d, y, 1.0), y);
    const double r = fmx(fmx(-d, y, 1.0), y, y);
    Coef<double> k;
    k.c1 = mk2((1.0 - t2) * r, -((2.0 * th) * r));
    k.c2 = mk2(r, -(th * r));
    return k;
}

// Per-site coefficients as kept in registers: complex64 the record gamma;
// complex128 alpha and Re beta, Im beta being half of Im alpha exactly.
template <typename R> struct T2Site;
template <> struct T2Site<float> {
    float2 g;
    __device__ __forceinline__ void load(const float *th, size_t idx, float sgn) {
        const float2 r = ((const float2 *)th)[idx];
        g = mk2(r.x, sgn * r.y);
    }
    __device__ __forceinline__ Coef<float> coef() const { return coef_site(g, 1.0f); }
};
template <> struct T2Site<double> {
    double2 c1;
    double c2x;
    __device__ __forceinline__ void load(const double *th, size_t idx, double sgn) {
        const Coef<double> k = coef_theta_r(sgn * th[idx]);
        c1 = k.c1;
        c2x = k.c2.x;
    }
    __device__ __forceinline__ Coef<double> coef() const {
        Coef<double> k;
        k.c1 = c1;
        k.c2 = mk2(c2x, 0.5 * c1.y);
        return k;
    }
};

// The exchange rows of one workgroup.
template <typename R, int NW> struct T2Edge {
    cx<R> e[2][2][NW][64];        // half-step parity; 0: first row, 1: last row; wave; lane
};

// steps: full steps of this pass (<= ring); (tx, ty): tile of (64 - 2 ring) x
// (NW K - 2 ring) cells.
template <typename R, bool SITE, bool ZB, int K, int NW>
__device__ __forceinline__ void tile2(const FusedArgs<R> &a, const R *__restrict__ tab, int steps, int ring, int tx,
                                      int ty, T2Edge<R, NW> &sh) {
    using C = cx<R>;
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nx = a.nx, ny = a.ny;
    const int tw = 64 - 2 * ring, th = NW * K - 2 * ring;
    const int x0 = tx * tw, y0 = ty * th;
    const int xl = x0 - ring + lane, yl = y0 - ring + wv * K;      // lattice position of this thread's first cell
    const bool inx = !ZB || (xl >= 0 && xl < nx);
    const int gx = ZB ? (inx ? xl : 0) : wrapn(xl, nx);
    const R rx = a.rx, ry = a.ry;
    const R sgn = a.rev ? (R)-1 : (R)1;

    C u0[K], u1[K], v0[K], v1[K];
    T2Site<R> s0[SITE ? K : 1], s1[SITE ? K : 1], s2[SITE ? K : 1], s3[SITE ? K : 1];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int y = yl + k;
        const bool iny = !ZB || (y >= 0 && y < ny);
        const size_t c = (size_t)(ZB ? (iny ? y : 0) : wrapn(y, ny)) * (size_t)nx + gx;
        u0[k] = ld_or0((const C *)a.in[0], c, inx && iny);
        u1[k] = ld_or0((const C *)a.in[1], c, inx && iny);
        v0[k] = ld_or0((const C *)a.in[2], c, inx && iny);
        v1[k] = ld_or0((const C *)a.in[3], c, inx && iny);
        if constexpr (SITE) {
            s0[k].load(a.th[0], c, sgn);
            s1[k].load(a.th[1], c, sgn);
            s2[k].load(a.th[2], c, sgn);
            s3[k].load(a.th[3], c, sgn);
        }
    }
    Coef<R> ku{}, kv{};
    if constexpr (!SITE) {
        const R *e = tab, *f = tab + 12;                            // classes 0 (u) and 3 (v), one plane
        ku.c1 = mk2(e[0], e[1]);
        ku.c2 = mk2(e[2], e[3]);
        kv.c1 = mk2(f[0], f[1]);
        kv.c2 = mk2(f[2], f[3]);
    }
    auto keep = [&](C &x, C v, int k) __attribute__((always_inline)) {
        if constexpr (ZB) {
            const int y = yl + k;
            const bool in = inx && y >= 0 && y < ny;
            x = mk2(in ? v.x : (R)0, in ? v.y : (R)0);
        } else {
            x = v;
        }
    };
    const int wa = min(wv + 1, NW - 1), wb = max(wv - 1, 0);
    // After lo full steps only rows lo .. NW K - 1 - lo of the region still matter:
    // a wave with none of them skips the half-step (not its barrier).
    const int r0 = wv * K;
    auto rows = [&](int lo, auto row) __attribute__((always_inline)) {
        if (r0 + K - 1 >= lo && r0 <= NW * K - 1 - lo) {
#pragma unroll
            for (int k = 0; k < K; ++k) row(k);
        }
    };
    auto half_u = [&](int lo) __attribute__((always_inline)) {
        sh.e[0][0][wv][lane] = v0[0];
        sh.e[0][1][wv][lane] = v1[K - 1];
        __syncthreads();
        const C up = sh.e[0][0][wa][lane], dn = sh.e[0][1][wb][lane];
        auto row = [&](int k) __attribute__((always_inline)) {
            const St2<C> s = stencil_u<C, R>(rx, ry, v0[k], t2_cxm(v0[k]), k + 1 < K ? v0[k + 1 < K ? k + 1 : 0] : up,
                                             v1[k], k > 0 ? v1[k > 0 ? k - 1 : 0] : dn, t2_cxp(v1[k]));
            keep(u0[k], update(u0[k], s.s0, SITE ? s0[SITE ? k : 0].coef() : ku), k);
            keep(u1[k], update(u1[k], s.s1, SITE ? s1[SITE ? k : 0].coef() : ku), k);
        };
        rows(lo, row);
    };
    auto half_v = [&](int lo) __attribute__((always_inline)) {
        sh.e[1][0][wv][lane] = u0[0];
        sh.e[1][1][wv][lane] = u1[K - 1];
        __syncthreads();
        const C up = sh.e[1][0][wa][lane], dn = sh.e[1][1][wb][lane];
        auto row = [&](int k) __attribute__((always_inline)) {
            const St2<C> s = stencil_v<C, R>(rx, ry, u0[k], t2_cxp(u0[k]), k + 1 < K ? u0[k + 1 < K ? k + 1 : 0] : up,
                                             u1[k], k > 0 ? u1[k > 0 ? k - 1 : 0] : dn, t2_cxm(u1[k]));
            keep(v0[k], update(v0[k], s.s0, SITE ? s2[SITE ? k : 0].coef() : kv), k);
            keep(v1[k], update(v1[k], s.s1, SITE ? s3[SITE ? k : 0].coef() : kv), k);
        };
        rows(lo, row);
    };
    // forward: (u v) x steps; reversed: v (u v) x (steps - 1) u
    const int s_end = a.rev ? steps + 1 : steps;
    for (int s = 0; s < s_end; ++s) {
        if (!a.rev || s > 0) half_u(a.rev ? s - 1 : s);
        if (!a.rev || s < steps) half_v(s);
    }

    const int w = min(tw, nx - x0), h = min(th, ny - y0);
    if (lane >= ring && lane < ring + w) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int rr = wv * K + k;
            if (rr >= ring && rr < ring + h) {
                const size_t c = (size_t)(yl + k) * (size_t)nx + xl;
                st_nt((C *)a.out[0] + c, u0[k]);
                st_nt((C *)a.out[1] + c, u1[k]);
                st_nt((C *)a.out[2] + c, v0[k]);
                st_nt((C *)a.out[3] + c, v1[k]);
            }
        }
    }
}

}  // namespace dirac
