// (2+1)D with gauge links: several steps per pass on the register tile of tile2.h.
//
// A cell keeps its eight link factors next to its amplitudes, so they cross the bus
// once per pass instead of once per step.  A u row multiplies each neighbour by its
// link; a v row takes conj(link) times the new u value, a product that only the u
// cell can form: the two that point across x go to the next lane, u1's +y product of
// a wave's last row and u0's -y product of its first row through LDS.  Same helpers
// and order as the one-step march (k2_fused_links), same bits.  Measured per step
// next to it, complex64, no potential: 64 x 64 1.4 against 13.2 us, 512 x 512 3.5
// against 21.9, 2048 x 2048 49 against 123; complex128 per site 2048 x 2048 111 against
// 300.
#include "gauge2.h"
#include "tile2.h"
#include "tile2_plan.h"

namespace dirac {

namespace {

template <typename R, bool SITE, int K, int NW>
__global__ __launch_bounds__(NW * 64, 4) void k2_tile_links(FusedArgs<R> a, LinkPtrs L, const R *__restrict__ tab,
                                                            int steps) {
    using C = cx<R>;
    __shared__ T2Edge<R, NW> sh;
    const int nb = gridDim.x, b = blockIdx.x, x = b & 7, bq = nb >> 3, br = nb & 7;
    const int tile = x * bq + min(x, br) + (b >> 3), tx = tile % a.ntx, ty = tile / a.ntx;
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nx = a.nx, ny = a.ny, ring = steps;
    const int tw = 64 - 2 * ring, th = NW * K - 2 * ring;
    const int x0 = tx * tw, y0 = ty * th;
    const int xl = x0 - ring + lane, yl = y0 - ring + wv * K;
    const R rx = a.rx, ry = a.ry;

    C u0[K], u1[K], v0[K], v1[K], l0[K][4], l1[K][4];
    T2Site<R> s0[SITE ? K : 1], s1[SITE ? K : 1], s2[SITE ? K : 1], s3[SITE ? K : 1];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const size_t c = (size_t)wrapn(yl + k, ny) * (size_t)nx + wrapn(xl, nx);
        u0[k] = ((const C *)a.in[0])[c];
        u1[k] = ((const C *)a.in[1])[c];
        v0[k] = ((const C *)a.in[2])[c];
        v1[k] = ((const C *)a.in[3])[c];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            l0[k][t] = ((const C *)L.u[t])[c];
            l1[k][t] = ((const C *)L.u[4 + t])[c];
        }
        if constexpr (SITE) {
            s0[k].load(a.th[0], c, (R)1);
            s1[k].load(a.th[1], c, (R)1);
            s2[k].load(a.th[2], c, (R)1);
            s3[k].load(a.th[3], c, (R)1);
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
    const int wa = min(wv + 1, NW - 1), wb = max(wv - 1, 0), r0 = wv * K;
    for (int s = 0; s < steps; ++s) {
        const bool live = r0 + K - 1 >= s && r0 <= NW * K - 1 - s;  // rows that still matter
        sh.e[0][0][wv][lane] = v0[0];
        sh.e[0][1][wv][lane] = v1[K - 1];
        __syncthreads();
        if (live) {
            const C up = sh.e[0][0][wa][lane], dn = sh.e[0][1][wb][lane];
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const C v0yp = k + 1 < K ? v0[k + 1 < K ? k + 1 : 0] : up, v1ym = k > 0 ? v1[k > 0 ? k - 1 : 0] : dn;
                u0[k] = update(u0[k], u_row0(l0[k], v0[k], t2_cxm(v0[k]), v1[k], v1ym, rx, ry),
                               SITE ? s0[SITE ? k : 0].coef() : ku);
                u1[k] = update(u1[k], u_row1(l1[k], t2_cxp(v1[k]), v1[k], v0yp, v0[k], rx, ry),
                               SITE ? s1[SITE ? k : 0].coef() : ku);
            }
        }
        sh.e[1][0][wv][lane] = pr(l0[0][T2YM], u0[0]);
        sh.e[1][1][wv][lane] = pr(l1[K - 1][T2YP], u1[K - 1]);
        __syncthreads();
        if (live) {
            const C up = sh.e[1][0][wa][lane], dn = sh.e[1][1][wb][lane];
            C below = dn;                                           // u1's +y product of the row below
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const C above = k + 1 < K ? pr(l0[k + 1 < K ? k + 1 : 0][T2YM], u0[k + 1 < K ? k + 1 : 0]) : up;
                const C T[8] = {t2_cxp(pr(l0[k][T2XM], u0[k])), pr(l0[k][T2XP], u0[k]), pr(l1[k][T2YM], u1[k]), below,
                                pr(l1[k][T2XM], u1[k]), t2_cxm(pr(l1[k][T2XP], u1[k])), above, pr(l0[k][T2YP], u0[k])};
                below = pr(l1[k][T2YP], u1[k]);
                const St2<C> S = v_rows(T, rx, ry);
                v0[k] = update(v0[k], S.s0, SITE ? s2[SITE ? k : 0].coef() : kv);
                v1[k] = update(v1[k], S.s1, SITE ? s3[SITE ? k : 0].coef() : kv);
            }
        }
    }
    const int w = min(tw, nx - x0), h = min(th, ny - y0);
    if (lane >= ring && lane < ring + w) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int rr = r0 + k;
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

}  // namespace

template <typename R>
hipError_t launch_tile2_links(const FusedArgs<R> &a0, const LinkPtrs &L, bool site, int steps, hipStream_t s) {
    FusedArgs<R> a = a0;
    if (steps < 1 || steps > kTile2MaxSteps || (!site && a.tab == nullptr)) return hipErrorInvalidValue;
    const int64_t nx = a.nx, ny = a.ny;
    double us = 0.0;
    const int shape = tile2_best_shape(steps, 1, &nx, &ny, sizeof(R) == 4, tile2_kind(site, true), &us);
    if (shape < 0) return hipErrorInvalidValue;
    const int64_t tiles = tile2_tiles(shape, steps, nx, ny);
    if (tiles > 0x7fffffff) return hipErrorInvalidValue;
    a.ntx = (a.nx + 64 - 2 * steps - 1) / (64 - 2 * steps);
    const dim3 g((unsigned)tiles), b(1024);
    if (shape == 0) {
        if (site) hipLaunchKernelGGL((k2_tile_links<R, true, 1, 16>), g, b, 0, s, a, L, a.tab, steps);
        else hipLaunchKernelGGL((k2_tile_links<R, false, 1, 16>), g, b, 0, s, a, L, a.tab, steps);
    } else if constexpr (sizeof(R) == 4) {
        if (site) hipLaunchKernelGGL((k2_tile_links<R, true, 2, 16>), g, b, 0, s, a, L, a.tab, steps);
        else hipLaunchKernelGGL((k2_tile_links<R, false, 2, 16>), g, b, 0, s, a, L, a.tab, steps);
    }
    return hipGetLastError();
}
template hipError_t launch_tile2_links<float>(const FusedArgs<float> &, const LinkPtrs &, bool, int, hipStream_t);
template hipError_t launch_tile2_links<double>(const FusedArgs<double> &, const LinkPtrs &, bool, int, hipStream_t);

}  // namespace dirac
