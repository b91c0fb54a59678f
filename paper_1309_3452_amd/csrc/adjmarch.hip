// One backward step of the adjoint per launch, as a z-march in registers.
//
// A backward step is sweep 1 on A,B (psi rebuilt, lam updated) and sweep 3 on C,D
// (lam updated, psi of the next step rebuilt), see adjoint.hip.  On the chain of
// half-planes along z (march3r.h) both are one update of the first field, then one
// of the second, each from the other at g-1, g, g+1: the same pipeline of two levels,
// one half-plane apart, with psi and lam side by side.  lam enters a stencil times
// conj(beta) (sweep 1) or beta (sweep 3) of its own plane, which is formed once per
// value.  As in place the two sweeps move 48 array passes a step (54 by the byte
// counters), here 32; the price is a second buffer set for lam.
//
// Same layout as the forward march: lane = column, a wave owns K rows, x neighbours by
// DPP shifts, wave-edge rows through double-buffered LDS, one barrier per iteration.
// The gradient's products of half-plane g come from level 1 at iteration g+1 and
// level 2 at g+2; a wave adds them up (DPP), lane 63 leaves the sum in LDS and after the
// barrier one thread adds the waves' sums in order and adds the result to the tile's
// slot, which no other workgroup touches in the launch.
#include <algorithm>
#include <type_traits>

#include "adjmarch.h"
#include "march2.h"
#include "march3r_plan.h"
#include "ntstore.h"
#include "stencil3.h"
#include "tile2.h"

namespace dirac {

namespace {

// Sum over the wave, in lane 63 (row shifts, then the row sums handed on).
template <int CTRL, int ROWS> __device__ __forceinline__ double dpp_add(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xf, false);
    return v + __hiloint2double(hi, lo);
}
__device__ __forceinline__ double wave_sum63(double v) {
    v = dpp_add<0x111, 0xf>(v);        // row_shr:1
    v = dpp_add<0x112, 0xf>(v);        // row_shr:2
    v = dpp_add<0x114, 0xf>(v);        // row_shr:4
    v = dpp_add<0x118, 0xf>(v);        // row_shr:8
    v = dpp_add<0x142, 0xa>(v);        // row_bcast:15 into rows 1 and 3
    return dpp_add<0x143, 0xc>(v);     // row_bcast:31 into rows 2 and 3
}

template <typename R, int K, int NW, int WPE, bool LAST>
__global__ __launch_bounds__(NW * 64, WPE) void k3_adj_march(AdjMarchArgs<R> a, const R *__restrict__ tab_f,
                                                             const R *__restrict__ tab_r, int tw) {
    using C = cx<R>;
    constexpr uint32_t CS = sizeof(C);
    constexpr int th = NW * K - 2;
    __shared__ C e[2 * 2 * 2 * 2 * NW * 64];
    __shared__ double red[2][NW];
    const int nb = gridDim.x, b = blockIdx.x, bx = b & 7, bq = nb >> 3, br_ = nb & 7;
    const int L = bx * bq + min(bx, br_) + (b >> 3);
    const int tx = L % a.ntx, ty = L / a.ntx % a.nty, zc = L / (a.ntx * a.nty);
    const int z0 = zc * a.zchunk, z1 = min(a.nz, z0 + a.zchunk);
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const int rg = (64 - tw) / 2, x0 = tx * tw, y0 = ty * th;
    const int w = min(tw, nx - x0), h = min(th, ny - y0);
    const int xl = x0 - rg + lane, yl = y0 - 1 + wv * K;
    const uint32_t pbytes = (uint32_t)nx * (uint32_t)ny * CS, tstride = (uint32_t)nz * (uint32_t)(4 * sizeof(R));
    uint32_t go[K];
    bool own[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int rr = wv * K + k;
        own[k] = lane >= rg && lane < rg + w && rr >= 1 && rr < 1 + h;
        go[k] = ((uint32_t)wrapn(yl + k, ny) * (uint32_t)nx + (uint32_t)wrapn(xl, nx)) * CS;
    }
    const R rx = a.rx, ry = a.ry, rz = a.rz;
    const C zero = mk2((R)0, (R)0);
    const int wa = min(wv + 1, NW - 1), wb = max(wv - 1, 0);
    // [buffer][level][first row's component 0, last row's component 1][psi, lam][wave][lane]
    auto edge = [&](int buf, int l, int c, int q, int wave) -> C & {
        return e[((((buf * 2 + l) * 2 + c) * 2 + q) * NW + wave) * 64 + lane];
    };
    int kr = z0 - 1, kw = wrapn(kr, nz);
    const int dm[3] = {0, 1 % nz, 2 % nz};
    auto stored = [&](int d) __attribute__((always_inline)) -> int {       // plane kr - d, wrapped
        if (d < 0) return kw + 1 == nz ? 0 : kw + 1;
        const int k = kw - dm[d < 0 ? 0 : d];
        return k < 0 ? k + nz : k;
    };
    auto coef = [&](const R *tab, int cls, int k) __attribute__((always_inline)) {
        const R *t = (const R *)((const char *)tab + (uint32_t)cls * tstride + (uint32_t)k * (uint32_t)(4 * sizeof(R)));
        Coef<R> q;
        q.c1 = mk2(t[0], t[1]);
        q.c2 = mk2(t[2], t[3]);
        return q;
    };

    // windows [half-plane mod 3][psi, factor times lam][component][row]: level 0 the
    // second field, level 1 the new first field; the second field's own lam
    C W[2][3][2][2][K], ly[3][2][K];
    C fo[2][2][K], sn[2][2][K], fn[2][2][K];            // [psi, lam][component][row]
#pragma unroll
    for (int l = 0; l < 2; ++l)
#pragma unroll
        for (int s = 0; s < 3; ++s)
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int c = 0; c < 2; ++c)
#pragma unroll
                    for (int k = 0; k < K; ++k) {
                        W[l][s][q][c][k] = zero;
                        if (l == 0 && q == 0) ly[s][c][k] = zero;
                    }
    double g1 = 0.0;                                     // level 1's products of half-plane h - 1
    const int hs = 2 * (z0 - 1), he = 2 * z1 + 1;

    auto load = [&](auto EV, auto DS, auto DF) __attribute__((always_inline)) {
        constexpr bool ev = decltype(EV)::value;
        const size_t ps = (size_t)(uint32_t)stored(decltype(DS)::value) * pbytes;
        const size_t pf = (size_t)(uint32_t)stored(decltype(DF)::value) * pbytes;
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int k = 0; k < K; ++k) {
                sn[0][c][k] = *(const C *)((const char *)a.f[(ev ? 6 : 4) + c] + ps + go[k]);
                sn[1][c][k] = *(const C *)((const char *)a.lam[(ev ? 6 : 4) + c] + ps + go[k]);
                fn[0][c][k] = *(const C *)((const char *)a.f[(ev ? 2 : 0) + c] + pf + go[k]);
                fn[1][c][k] = *(const C *)((const char *)a.lam[(ev ? 2 : 0) + c] + pf + go[k]);
            }
    };
    double *slot = a.gpart + (size_t)(tx + a.ntx * ty) * (size_t)nz * 2;
    // the waves' sums of half-plane g, left in LDS by the iteration before
    auto add_grad = [&](int buf, int g) __attribute__((always_inline)) {
        if (threadIdx.x == 0 && g >= 2 * z0) {
            double s = red[buf][0];
#pragma unroll
            for (int v = 1; v < NW; ++v) s += red[buf][v];
            unsafeAtomicAdd(slot + g, s);                 // [plane][integer z, half-integer z]
        }
    };

    auto iter = [&](auto PH, auto FILL, int hh) __attribute__((always_inline)) {
        constexpr int ph = decltype(PH)::value;
        constexpr int fill = decltype(FILL)::value ? ph / 2 : 2;
        constexpr int bw = ph & 1, br = bw ^ 1;
        if constexpr (!decltype(FILL)::value || ph > 4) add_grad(br, hh - 3);
        const Coef<R> kb = coef(tab_f, (ph & 1) ? 2 : 3, stored(0));
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int k = 0; k < K; ++k) {
                W[0][ph % 3][0][c][k] = sn[0][c][k];
                W[0][ph % 3][1][c][k] = cmulc(kb.c2, sn[1][c][k]);
                ly[ph % 3][c][k] = sn[1][c][k];
                fo[0][c][k] = fn[0][c][k];
                fo[1][c][k] = fn[1][c][k];
            }
#pragma unroll
        for (int k = 0; k < K; ++k) asm volatile("" : "+v"(go[k]));
        if (hh < he)
            load(std::integral_constant<bool, (ph & 1) == 1>(), std::integral_constant<int, (ph & 1) ? -1 : 0>(),
                 std::integral_constant<int, 0>());
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            edge(bw, 0, 0, q, wv) = W[0][ph % 3][q][0][0];
            edge(bw, 0, 1, q, wv) = W[0][ph % 3][q][1][K - 1];
        }
        double gsum = g1;                                // of half-plane hh - 2
        auto level = [&](auto LV) __attribute__((always_inline)) {
            constexpr int l = decltype(LV)::value;
            constexpr bool first = l == 1;
            constexpr bool geven = ((ph + l) & 1) == 0;
            constexpr bool rowP = first == geven;
            constexpr int sp = (ph + 18 - l + 1) % 3, sm = (ph + 18 - l) % 3, so = (ph + 18 - l - 1) % 3;
            constexpr int d = (l - (ph & 1) + 1) / 2;
            const int g = hh - l;
            const bool st = g >= 2 * z0 && g < 2 * z1;
            const size_t po = (size_t)(uint32_t)(kr - d) * pbytes;
            const int cls = first ? (geven ? 0 : 1) : (geven ? 3 : 2), kp = stored(d);
            const Coef<R> kf = coef(tab_f, cls, kp), kv = coef(tab_r, cls, kp);
            C S[2][2][K];                                // [psi, lam]: the stencils
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const C up = edge(br, l - 1, 0, q, wa), dn = edge(br, l - 1, 1, q, wb);
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    const C m0 = W[l - 1][sm][q][0][k], m1 = W[l - 1][sm][q][1][k];
                    const C dz0 = csub(W[l - 1][sp][q][0][k], W[l - 1][so][q][0][k]);
                    const C dz1 = csub(W[l - 1][sp][q][1][k], W[l - 1][so][q][1][k]);
                    const C m1ym = k > 0 ? W[l - 1][sm][q][1][k > 0 ? k - 1 : 0] : dn;
                    const C m0yp = k + 1 < K ? W[l - 1][sm][q][0][k + 1 < K ? k + 1 : 0] : up;
                    if constexpr (rowP) {
                        S[q][0][k] = sterm3(rz, dz0, rx, csub(m0, t2_cxm(m0)), -ry, csub(m1, m1ym));
                        S[q][1][k] = sterm3(rz, dz1, rx, csub(t2_cxp(m1), m1), -ry, csub(m0yp, m0));
                    } else {
                        S[q][0][k] = sterm3(-rz, dz0, rx, csub(t2_cxp(m0), m0), ry, csub(m1, m1ym));
                        S[q][1][k] = sterm3(-rz, dz1, rx, csub(m1, t2_cxm(m1)), ry, csub(m0yp, m0));
                    }
                }
            }
            double gl = 0.0;
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    const C old = first ? fo[0][c][k] : W[0][sm][0][c][k];
                    const C neg = mk2(-S[0][c][k].x, -S[0][c][k].y);
                    C nw = old, ln;
                    if constexpr (first) {
                        const C lx = cadd(fo[1][c][k], S[1][c][k]);
                        nw = update(old, neg, kv);
                        if (st && own[k]) gl += dtheta_term(lx, old, nw, kf);
                        ln = cmulc(alpha_of(kf), lx);
                        W[1][sm][0][c][k] = nw;
                        W[1][sm][1][c][k] = cmul(kf.c2, ln);
                    } else {
                        ln = cadd(cmulc(alpha_of(kf), ly[sm][c][k]), S[1][c][k]);
                        if constexpr (!LAST) {
                            nw = update(old, neg, kv);
                            if (st && own[k]) gl += dtheta_term(ln, old, nw, kf);
                        }
                    }
                    if (st && own[k]) {
                        constexpr int arr = first ? (geven ? 0 : 2) : (geven ? 6 : 4);
                        st_nt((C *)((char *)a.fo[arr + c] + po + go[k]), nw);
                        st_nt((C *)((char *)a.lamo[arr + c] + po + go[k]), ln);
                    }
                }
            if constexpr (first) {
                g1 = gl;
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    edge(bw, 1, 0, q, wv) = W[1][sm][q][0][0];
                    edge(bw, 1, 1, q, wv) = W[1][sm][q][1][K - 1];
                }
            } else {
                gsum += gl;
            }
        };
        if constexpr (fill >= 1) level(std::integral_constant<int, 1>());
        if constexpr (fill >= 2) level(std::integral_constant<int, 2>());
        if constexpr (!decltype(FILL)::value || ph >= 4) {
            gsum = wave_sum63(gsum);
            if (lane == 63) red[bw][wv] = gsum;
        }
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if constexpr (ph & 1) {
            ++kr;
            kw = kw + 1 == nz ? 0 : kw + 1;
        }
    };

    load(std::integral_constant<bool, true>(), std::integral_constant<int, 0>(), std::integral_constant<int, 1>());
    constexpr std::true_type filling{};
    constexpr std::false_type full{};
    iter(std::integral_constant<int, 0>(), filling, hs);
    iter(std::integral_constant<int, 1>(), filling, hs + 1);
    iter(std::integral_constant<int, 2>(), filling, hs + 2);
    iter(std::integral_constant<int, 3>(), filling, hs + 3);
    iter(std::integral_constant<int, 4>(), filling, hs + 4);
    iter(std::integral_constant<int, 5>(), filling, hs + 5);
    for (int hh = hs + 6; hh <= he; hh += 6) {
        iter(std::integral_constant<int, 0>(), full, hh);
        iter(std::integral_constant<int, 1>(), full, hh + 1);
        if (hh + 2 > he) break;
        iter(std::integral_constant<int, 2>(), full, hh + 2);
        iter(std::integral_constant<int, 3>(), full, hh + 3);
        if (hh + 4 > he) break;
        iter(std::integral_constant<int, 4>(), full, hh + 4);
        iter(std::integral_constant<int, 5>(), full, hh + 5);
    }
    add_grad(1, he - 2);                                 // he - hs is odd
}

constexpr int kAdjRows = 14, kAdjRows64 = 6;             // tile rows, complex64 and complex128

int adj_width(int nx) { return (nx + 61) / 62 < (nx + 55) / 56 && nx <= 280 ? 62 : 56; }

}  // namespace

int adj_march_tiles(int nx, int ny) {
    return ((nx + adj_width(nx) - 1) / adj_width(nx)) * ((ny + kAdjRows64 - 1) / kAdjRows64);
}

// A march iteration takes about 3.4 us (complex128; complex64 4.6, with twice the
// rows), the sweeps move psi and lam three times at 5.6 (6.3) TB/s out of the caches
// and 4.8 (4.0) from HBM.  Measured per backward step, in place / march: complex128
// 64^3 40 / 46 us, 96^3 126 / 109, 128^3 308 / 287, 200 x 168 x 152 890 / 604, 256^3
// 2560 / 1861; complex64 64^3 23 / 32, 128^3 127 / 158 (three tiles of 56 for 128
// columns), 200 x 168 x 152 548 / 315, 256^3 1546 / 1029.
bool adj_march_wins(bool fp32, int nx, int ny, int nz) {
    const int tw = adj_width(nx), th = fp32 ? kAdjRows : kAdjRows64;
    const int64_t tiles = (int64_t)((nx + tw - 1) / tw) * ((ny + th - 1) / th), cus = resident_per_round();
    const int nzc = pick_chunks(tiles, nz, 1);
    const double march = 4.0 + (double)((tiles * nzc + cus - 1) / cus) * 2.0 * ((nz + nzc - 1) / nzc + 1) *
                                   (fp32 ? 4.6 : 3.4);
    const double bytes = (double)nx * ny * nz * (fp32 ? 128.0 : 256.0);
    const double rate = bytes < 3e8 ? (fp32 ? 6.3e6 : 5.6e6) : (fp32 ? 4.0e6 : 4.8e6);
    return march < std::max(11.5, 3.0 * bytes / rate);
}

template <typename R>
hipError_t launch_adj_march(const AdjMarchArgs<R> &a0, const R *tab_f, const R *tab_r, bool last, hipStream_t s) {
    AdjMarchArgs<R> a = a0;
    constexpr bool fp32 = sizeof(R) == 4;
    constexpr int K = 1, NW = fp32 ? 16 : 8, WPE = fp32 ? 4 : 2;
    const int tw = adj_width(a.nx), th = fp32 ? kAdjRows : kAdjRows64;
    if ((uint64_t)a.nx * (uint64_t)a.ny * sizeof(cx<R>) >= (1ull << 32)) return hipErrorInvalidValue;
    a.ntx = (a.nx + tw - 1) / tw;
    a.nty = (a.ny + th - 1) / th;
    const int nzc = pick_chunks((int64_t)a.ntx * a.nty, a.nz, 1);
    a.zchunk = (a.nz + nzc - 1) / nzc;
    const int64_t nblk = (int64_t)a.ntx * a.nty * ((a.nz + a.zchunk - 1) / a.zchunk);
    if (nblk > 0x7fffffff) return hipErrorInvalidValue;
    const dim3 g((unsigned)nblk), b(NW * 64);
    if (last) hipLaunchKernelGGL((k3_adj_march<R, K, NW, WPE, true>), g, b, 0, s, a, tab_f, tab_r, tw);
    else hipLaunchKernelGGL((k3_adj_march<R, K, NW, WPE, false>), g, b, 0, s, a, tab_f, tab_r, tw);
    return hipGetLastError();
}
template hipError_t launch_adj_march<float>(const AdjMarchArgs<float> &, const float *, const float *, bool, hipStream_t);
template hipError_t launch_adj_march<double>(const AdjMarchArgs<double> &, const double *, const double *, bool,
                                             hipStream_t);

}  // namespace dirac
