// (3+1)D: T time steps per launch as a z-march that lives in registers (Sect. 2,
// Eqs. ss1-ss4).
//
// Along z the grid of Eq. (ABCDgrid) is a chain of half-planes: half-plane 2k
// (z = k) holds A and D of plane k, half-plane 2k+1 (z = k + 1/2) B and C.  On
// each, A or B is the first field of a step and D or C the second; the update of
// the first field at half-plane g takes the second field at g-1, g, g+1 and the
// other way round, so one kind of row serves all four equations.  With level 0
// the old second field and level l (1 .. 2T) the fields after half-step l, the
// march runs all levels as a pipeline, each one half-plane behind the previous:
// iteration h loads half-plane h and evaluates level l at g = h - l from level
// l-1 at g+1 (just computed), g and g-1, and from the old value level l-2 at g.
// So of every level only the last three half-planes are alive, and only at the
// thread's own cells.
//
// A workgroup of NW waves covers 64 x (NW K) cells of x and y: the tile plus a
// ring of T cells on each side, recomputed (a wrong value at the rim moves one
// cell inwards per step).  Lane l of wave w owns column l of rows w K .. w K +
// K - 1.  x neighbours come from the next lane by a DPP wave shift, y neighbours
// inside the thread's rows from its own registers; only the first row's component
// 0 and the last row's component 1 of each level go through LDS.  The y neighbours
// lie on half-plane g, computed one iteration earlier, so one barrier per
// iteration (double-buffered edges) serves all levels.  The loop is unrolled by
// six: windows rotate by three, the kind of half-plane and the LDS buffer by two,
// and no value is ever moved.  The next half-plane's loads are issued at the top
// of an iteration and land during it; the barrier waits for LDS only.
//
// The helpers and operation order are those of the other kernels: same bits.
#pragma once

#include <algorithm>
#include <iterator>
#include <type_traits>

#include "device.h"
#include "internal.h"
#include "march2.h"
#include "march3r_plan.h"
#include "ntstore.h"
#include "stencil3.h"
#include "tile2.h"

namespace dirac {

template <typename R> struct M3Rec;
template <> struct M3Rec<float> {
    typedef float2 T;
    template <int SITE> static __device__ __forceinline__ Coef<float> coef(T g) {
        return coef_site(g, SITE == 2 ? -1.0f : 1.0f);
    }
};
template <> struct M3Rec<double> {
    typedef double T;
    template <int SITE> static __device__ __forceinline__ Coef<double> coef(T th) {
        return coef_theta_r(SITE == 2 ? -th : th);
    }
};

// Twelve waves of complex128 rows would need 192 KB for double-buffered edges.  They
// take single ones and a second barrier, between levels 2 and 3: edges of levels 0
// and 1 are read before it and written after it, those of levels 2 and 3 read
// after it and written before it, in the next iteration.
template <typename R, int T, int K, int NW> constexpr bool m3_single() { return sizeof(R) == 8 && T == 2 && NW > 8; }
template <typename R, int T, int K, int NW> constexpr int m3_edges() {
    return (m3_single<R, T, K, NW>() ? 1 : 2) * 2 * T * 2 * NW * 64;
}

// z0, z1: planes of this workgroup; (tx, ty): its tile of tw x (NW K - 2T)
// cells, tw even and at most 64 - 2T.  SITE: 0 V(z) tables, 1 per-site records, 2
// records with theta -> -theta.  ZB: zero values outside the lattice (cells there
// hold zero on every level).  e: m3_edges complex values of LDS.  nrm:
// with NORM, this thread's sums of the functional (C,D-summed form) and the plain
// norm.  XP: nx divides 64, the wave holds whole periods of a row and its shifts
// rotate, so x takes no ring (one tile).  A plane is below 4 GiB.
template <typename R, int T, int K, int NW, int SITE, bool ZB, bool NORM, bool XP>
__device__ __forceinline__ void march3r(const FusedArgs<R> &a, const R *__restrict__ tab, int tw, int tx, int ty,
                                        int z0, int z1, cx<R> *e, double (&nrm)[2]) {
    using C = cx<R>;
    using Rec = typename M3Rec<R>::T;
    constexpr int NL = 2 * T;
    constexpr uint32_t CS = sizeof(C), RS = sizeof(Rec);
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nx = a.nx, ny = a.ny, nz = a.nz, zh = a.zh;
    constexpr int th = NW * K - 2 * T;
    const int rg = XP ? 0 : (64 - tw) / 2;
    const int x0 = tx * tw, y0 = ty * th;
    const int w = min(tw, nx - x0), h = min(th, ny - y0);
    const int xl = x0 - rg + lane, yl = y0 - T + wv * K;
    const bool inx = !ZB || (xl >= 0 && xl < nx);
    const uint32_t pbytes = (uint32_t)nx * (uint32_t)ny * CS, rbytes = (uint32_t)nx * (uint32_t)ny * RS;
    const uint32_t tstride = (uint32_t)(nz + 2 * zh) * (uint32_t)(4 * sizeof(R));
    uint32_t go[K];                         // byte offset of the cell within a plane
    bool in[K], own[K];                     // inside the lattice; in the tile
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int y = yl + k, rr = wv * K + k;
        in[k] = inx && (!ZB || (y >= 0 && y < ny));
        own[k] = lane >= rg && lane < rg + w && rr >= T && rr < T + h;
        const int gy = ZB ? (in[k] ? y : 0) : wrapn(y, ny), gx = ZB ? (in[k] ? xl : 0) : wrapn(xl, nx);
        go[k] = ((uint32_t)gy * (uint32_t)nx + (uint32_t)gx) * CS;
    }
    const R rx = a.rx, ry = a.ry, rz = a.rz;
    const C zero = mk2((R)0, (R)0);
    const int wa = min(wv + 1, NW - 1), wb = max(wv - 1, 0);
    constexpr bool SB = m3_single<R, T, K, NW>();
    auto edge = [&](int buf, int l, int c, int wave) -> C & {
        return e[((((SB ? 0 : buf) * NL + l) * 2 + c) * NW + wave) * 64 + lane];
    };
    // plane of half-plane h, as it is (kr) and among the stored ones (kw), advanced
    // along the march; stored index of plane kr - d.  A slab's planes, and those of a
    // lattice with zero values outside, end; what a level computes from planes beyond
    // them reaches no stored value, so any stored plane serves there.
    // Up to 16 rows (EARLY) an iteration is one block without branches, which the
    // compiler can schedule: planes wrap by selects, loads go out unconditionally (the
    // last ones unused), and the tables' coefficients are read an iteration ahead, as
    // scalar loads right before their use put four latencies into each iteration.  Two
    // steps of 64^3: complex64 17.5 -> 15.3 us, with records 20.7 -> 17.4; complex128
    // 22.7 -> 21.3, with records 28.0 -> 26.9, and 200 x 168 x 152 with records
    // 442 -> 413.  With 16 rows the levels are kept apart (moved into each other they
    // cost 191 x 151 x 127 139 us; apart 131, with the branches 135).  The masks that a
    // zero boundary needs then cost more than it gains (128^3 complex128: 129 -> 132).
    constexpr bool EARLY = K * NW <= 16 && !ZB, APART = EARLY && K * NW == 16;
    const int nzs = nz + 2 * zh;
    int kr = z0 - T, kw = EARLY ? wrapn(kr + zh, nzs) : wrapn(kr, nz);
    int dm[T + 2];
#pragma unroll
    for (int d = 0; d < T + 2; ++d) dm[d] = d % (EARLY ? nzs : nz);
    auto stored = [&](int d) __attribute__((always_inline)) -> int {
        if constexpr (EARLY) {
            const int k = d < 0 ? kw + 1 - nzs : kw - dm[d < 0 ? 0 : d];
            return k < 0 ? k + nzs : k;
        }
        if (zh) return min(max(kr - d + zh, 0), nzs - 1);
        if (d < 0) return kw + 1 == nz ? 0 : kw + 1;
        const int k = kw - dm[d < 0 ? 0 : d];
        return k < 0 ? k + nz : k;
    };
    auto inz = [&](int d) __attribute__((always_inline)) -> bool { return !ZB || (kr - d >= 0 && kr - d < nz); };

    C W[NL][3][2][K];                       // [level][half-plane mod 3][component][row]
    static_assert(SITE == 0 || T <= 2, "the record windows hold three half-planes");
    // records of the first, second field [half-plane mod 3]: each serves two levels
    // (loaded a second time for levels 3 and 4 they cost a third more time)
    Rec qf[SITE ? 3 : 1][2][SITE ? K : 1], qs[SITE ? 3 : 1][2][SITE ? K : 1];
    C fo[2][K], sn[2][K], fn[2][K];         // old first field of h-1; next iteration's second and first
    Rec qfn[2][SITE ? K : 1], qsn[2][SITE ? K : 1];
#pragma unroll
    for (int l = 0; l < NL; ++l)
#pragma unroll
        for (int s = 0; s < 3; ++s)
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int k = 0; k < K; ++k) W[l][s][c][k] = zero;
    if constexpr (SITE != 0)
        for (int s = 0; s < 3; ++s)
            for (int c = 0; c < 2; ++c)
                for (int k = 0; k < K; ++k) {
                    qf[s][c][k] = Rec{};
                    qs[s][c][k] = Rec{};
                }

    const int hs = 2 * (z0 - T), he = 2 * z1 - 1 + NL;
    // loads for iteration h: the old second field of half-plane h and the old
    // first field of h-1 (ev: h is even); the records of the first field at h-1
    // and of the second at h-2, where levels 1 and 2 use them.  ds, df, dq: their
    // planes behind kr.  what: 1 the second field (and records), 2 the first, 3 both.
    auto load = [&](auto EV, auto DS, auto DF, auto DQ, int what) __attribute__((always_inline)) {
        constexpr bool ev = decltype(EV)::value;
        constexpr int ds = decltype(DS)::value, df = decltype(DF)::value, dq = decltype(DQ)::value;
        const bool oks = inz(ds), okf = inz(df);
        const size_t ps = (size_t)(uint32_t)stored(ds) * pbytes, pf = (size_t)(uint32_t)stored(df) * pbytes;
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const char *bs = (const char *)a.in[(ev ? 6 : 4) + c] + ps, *bf = (const char *)a.in[(ev ? 2 : 0) + c] + pf;
                if constexpr (ZB) {
                    if (what & 1) {
                        sn[c][k] = zero;
                        if (oks && in[k]) sn[c][k] = *(const C *)(bs + go[k]);
                    }
                    if (what & 2) {
                        fn[c][k] = zero;
                        if (okf && in[k]) fn[c][k] = *(const C *)(bf + go[k]);
                    }
                } else {
                    if (what & 1) sn[c][k] = *(const C *)(bs + go[k]);
                    if (what & 2) fn[c][k] = *(const C *)(bf + go[k]);
                }
            }
        if constexpr (SITE != 0) {
            const size_t qpf = (size_t)(uint32_t)stored(df) * rbytes, qps = (size_t)(uint32_t)stored(dq) * rbytes;
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    const uint32_t ro = go[k] / (CS / RS);
                    qfn[c][k] = *(const Rec *)((const char *)a.th[(ev ? 2 : 0) + c] + qpf + ro);
                    qsn[c][k] = *(const Rec *)((const char *)a.th[(ev ? 6 : 4) + c] + qps + ro);
                }
        }
    };
    auto tcoef = [&](int cls, int k) __attribute__((always_inline)) {
        const R *t = (const R *)((const char *)tab + (uint32_t)cls * tstride + (uint32_t)k * (uint32_t)(4 * sizeof(R)));
        Coef<R> q;
        q.c1 = mk2(t[0], t[1]);
        q.c2 = mk2(t[2], t[3]);
        return q;
    };

    // the coefficients of this iteration, and those of the one after a phase PH
    constexpr bool AHEAD = EARLY && SITE == 0;
    Coef<R> kc[SITE ? 1 : NL];
    auto tables = [&](auto PH, Coef<R>(&q)[SITE ? 1 : NL]) __attribute__((always_inline)) {
        constexpr int ph = decltype(PH)::value;
        if constexpr (AHEAD)
#pragma unroll
            for (int l = 1; l <= NL; ++l) {
                const bool geven = ((ph + 1 + l) & 1) == 0;
                q[l - 1] = tcoef((l & 1) ? (geven ? 0 : 1) : (geven ? 3 : 2), stored((ph & 1) ? (l + 1) / 2 - 1 : l / 2));
            }
    };

    // iteration hh, hh - hs = PH (mod 6); FILL: hh - hs = PH, where level l has
    // nothing yet that a stored value depends on before iteration 2 l
    auto iter = [&](auto PH, auto FILL, int hh) __attribute__((always_inline)) {
        constexpr int ph = decltype(PH)::value;
        constexpr int fill = decltype(FILL)::value ? ph / 2 : 2 * T;         // levels evaluated
        constexpr int bw = ph & 1, br = bw ^ 1;
        // this iteration's inputs arrive in the windows
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int k = 0; k < K; ++k) {
                W[0][ph % 3][c][k] = sn[c][k];
                fo[c][k] = fn[c][k];
                if constexpr (SITE != 0) {
                    qf[(ph + 2) % 3][c][k] = qfn[c][k];
                    qs[(ph + 1) % 3][c][k] = qsn[c][k];
                }
            }
#pragma unroll
        for (int k = 0; k < K; ++k) asm volatile("" : "+v"(go[k]));
        // next, for h = 2k: C and A of plane k; for h = 2k+1: D of plane k+1, B of k.
        // With tables the first field's loads go out after level 2: spread over the
        // iteration they cost 2 to 6% less time than in one burst (256^3 complex64
        // 271 against 281 us per step; with records 17% more, so there they stay).
        auto next = [&](int what) __attribute__((always_inline)) {
            if (EARLY || hh < he)
                load(std::integral_constant<bool, (ph & 1) == 1>(), std::integral_constant<int, (ph & 1) ? -1 : 0>(),
                     std::integral_constant<int, 0>(), std::integral_constant<int, (ph & 1) ? 0 : 1>(), what);
        };
        next(SITE == 0 ? 1 : 3);
        // edges of level l's newest half-plane, of this iteration or (ago = 1) the last
        auto put = [&](auto LV, int ago) __attribute__((always_inline)) {
            constexpr int l = decltype(LV)::value;
            edge(bw, l, 0, wv) = W[l][(ph + 18 - l - ago) % 3][0][0];
            edge(bw, l, 1, wv) = W[l][(ph + 18 - l - ago) % 3][1][K - 1];
        };
        if constexpr (SB) {
            put(std::integral_constant<int, 2>(), 1);
            put(std::integral_constant<int, 3>(), 1);
        } else {
            put(std::integral_constant<int, 0>(), 0);
        }
        auto xm = [](C v) __attribute__((always_inline)) { return XP ? t2_rxm(v) : t2_cxm(v); };
        auto xp = [](C v) __attribute__((always_inline)) { return XP ? t2_rxp(v) : t2_cxp(v); };
        auto level = [&](auto LV) __attribute__((always_inline)) {
            constexpr int l = decltype(LV)::value;
            constexpr bool first = l & 1;                            // the first field (A, B)
            constexpr bool geven = ((ph + l) & 1) == 0;              // half-plane g = hh - l
            constexpr bool rowP = first == geven;                    // A and C rows; else B and D
            constexpr int sp = (ph + 18 - l + 1) % 3, sm = (ph + 18 - l) % 3, so = (ph + 18 - l - 1) % 3;
            constexpr int d = (l - (ph & 1) + 1) / 2;                // plane of g: kr - d
            const int g = hh - l;
            if constexpr (APART) __builtin_amdgcn_sched_barrier(0);
            const C up = edge(br, l - 1, 0, wa), dn = edge(br, l - 1, 1, wb);
            Coef<R> kt{};
            if constexpr (AHEAD) kt = kc[SITE ? 0 : l - 1];
            else if constexpr (SITE == 0) kt = tcoef(first ? (geven ? 0 : 1) : (geven ? 3 : 2), stored(d));
            const bool zin = inz(d);
            const bool st = l >= NL - 1 && g >= 2 * z0 && g < 2 * z1;
            const size_t po = (size_t)(uint32_t)(kr - d + zh) * pbytes;
            C o[2][K], S[2][K];
            // with zero values outside, the functional in complex64 takes its
            // differences in FP64, as the reduction over the state does
            constexpr bool wide = NORM && ZB && sizeof(R) == 4 && l == NL;
            double2 Sd[wide ? 2 : 1][wide ? K : 1];
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const C m0 = W[l - 1][sm][0][k], m1 = W[l - 1][sm][1][k];
                const C dz0 = csub(W[l - 1][sp][0][k], W[l - 1][so][0][k]);
                const C dz1 = csub(W[l - 1][sp][1][k], W[l - 1][so][1][k]);
                const C m1ym = k > 0 ? W[l - 1][sm][1][k > 0 ? k - 1 : 0] : dn;
                const C m0yp = k + 1 < K ? W[l - 1][sm][0][k + 1 < K ? k + 1 : 0] : up;
                if constexpr (rowP) {
                    S[0][k] = sterm3(rz, dz0, rx, csub(m0, xm(m0)), -ry, csub(m1, m1ym));
                    S[1][k] = sterm3(rz, dz1, rx, csub(xp(m1), m1), -ry, csub(m0yp, m0));
                } else {
                    S[0][k] = sterm3(-rz, dz0, rx, csub(xp(m0), m0), ry, csub(m1, m1ym));
                    S[1][k] = sterm3(-rz, dz1, rx, csub(m1, xm(m1)), ry, csub(m0yp, m0));
                }
                if constexpr (wide) {
                    auto d = [](C p, C q) { return make_double2((double)p.x - (double)q.x, (double)p.y - (double)q.y); };
                    const C *z0p = &W[l - 1][sp][0][k], *z0m = &W[l - 1][so][0][k];
                    const C *z1p = &W[l - 1][sp][1][k], *z1m = &W[l - 1][so][1][k];
                    const double dx = rx, dy = rowP ? -(double)ry : (double)ry, dz = rowP ? (double)rz : -(double)rz;
                    const C xa = rowP ? xm(m0) : xp(m0), xb = rowP ? xp(m1) : xm(m1);
                    Sd[0][wide ? k : 0] = sterm3(dz, d(*z0p, *z0m), dx, rowP ? d(m0, xa) : d(xa, m0), dy, d(m1, m1ym));
                    Sd[wide ? 1 : 0][wide ? k : 0] =
                        sterm3(dz, d(*z1p, *z1m), dx, rowP ? d(xb, m1) : d(m1, xb), dy, d(m0yp, m0));
                }
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    C old;
                    if constexpr (l == 1) old = fo[c][k];
                    else old = W[l >= 2 ? l - 2 : 0][sm][c][k];      // level l-2 at g: the oldest of its window
                    Coef<R> q = kt;
                    if constexpr (SITE != 0)
                        q = M3Rec<R>::template coef<SITE>(first ? qf[(ph + 18 - l) % 3][c][k] : qs[(ph + 18 - l) % 3][c][k]);
                    C v = update(old, S[c][k], q);
                    if constexpr (ZB) v = mk2(in[k] && zin ? v.x : (R)0, in[k] && zin ? v.y : (R)0);
                    o[c][k] = v;
                }
            }
            if constexpr (l < NL) {
                constexpr int sw = (ph + 18 - l) % 3;
#pragma unroll
                for (int c = 0; c < 2; ++c)
#pragma unroll
                    for (int k = 0; k < K; ++k) W[l < NL ? l : 0][sw][c][k] = o[c][k];
                if constexpr (!SB) put(std::integral_constant<int, (l < NL ? l : 0)>(), 0);
            }
            if constexpr (l >= NL - 1) {
                if (st) {
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        constexpr int arr = first ? (geven ? 0 : 2) : (geven ? 6 : 4);
                        char *b = (char *)a.out[arr + c] + po;
#pragma unroll
                        for (int k = 0; k < K; ++k)
                            if (own[k]) {
                                st_nt((C *)(b + go[k]), o[c][k]);
                                if constexpr (NORM) {
                                    const double yr = (double)o[c][k].x, yi = (double)o[c][k].y;
                                    const double pp = yr * yr + yi * yi;
                                    nrm[1] += pp;
                                    double sr = (double)S[c][k].x, si = (double)S[c][k].y;
                                    if constexpr (wide) {
                                        sr = Sd[wide ? c : 0][wide ? k : 0].x;
                                        si = Sd[wide ? c : 0][wide ? k : 0].y;
                                    }
                                    nrm[0] += first ? pp : pp + (yr * sr + yi * si);
                                }
                            }
                    }
                }
            }
        };
        if constexpr (fill >= 1) level(std::integral_constant<int, 1>());
        if constexpr (fill >= 2) level(std::integral_constant<int, 2>());
        if constexpr (SITE == 0) next(2);
        if constexpr (SB) {
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            put(std::integral_constant<int, 0>(), 0);
            put(std::integral_constant<int, 1>(), 0);
        }
        if constexpr (T > 1 && fill >= 3) level(std::integral_constant<int, (T > 1 ? 3 : 1)>());
        Coef<R> kn[SITE ? 1 : NL];
        tables(std::integral_constant<int, ph>(), kn);
        if constexpr (T > 1 && fill >= 4) level(std::integral_constant<int, (T > 1 ? 4 : 2)>());
        if constexpr (T > 2 && fill >= 5) level(std::integral_constant<int, (T > 2 ? 5 : 1)>());
        if constexpr (T > 2 && fill >= 6) level(std::integral_constant<int, (T > 2 ? 6 : 2)>());
        // the edges written, those of the previous iteration read: a barrier that
        // waits for this wave's LDS operations only (loads and stores stay in flight)
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if constexpr (AHEAD)
#pragma unroll
            for (int l = 0; l < NL; ++l) {
                asm volatile("" : "+s"(kn[l].c1.x), "+s"(kn[l].c1.y), "+s"(kn[l].c2.x), "+s"(kn[l].c2.y));
                kc[l] = kn[l];
            }
        if constexpr (ph & 1) {
            ++kr;
            kw = kw + 1 == (EARLY ? nzs : nz) ? 0 : kw + 1;
        }
    };

    // for h = hs = 2k: D of plane k, B of k-1
    load(std::integral_constant<bool, true>(), std::integral_constant<int, 0>(), std::integral_constant<int, 1>(),
         std::integral_constant<int, 1>(), 3);
    // phase -1's successor is iteration hs, one half-plane on
    if constexpr (AHEAD)
#pragma unroll
        for (int l = 1; l <= NL; ++l)
            kc[l - 1] = tcoef((l & 1) ? 1 : 3, stored((l + 1) / 2));
    // 2 (z1 - z0) + 4 T iterations: an even number, at least six
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
}

template <typename R, int T, int K, int NW, int WPE, int SITE, bool ZB, bool NORM, bool XP>
__global__ __launch_bounds__(NW * 64, WPE) void k3_march3r(FusedArgs<R> a, const R *__restrict__ tab, int tw) {
    __shared__ cx<R> e[m3_edges<R, T, K, NW>()];
    __shared__ double red[NORM ? 2 * NW : 1];
    // each XCD (blocks are dealt to the eight in turn) takes a contiguous run of tiles
    const int n = gridDim.x, b = blockIdx.x, x = b & 7, q = n >> 3, r = n & 7;
    const int L = x * q + min(x, r) + (b >> 3);
    const int tx = L % a.ntx, ty = L / a.ntx % a.nty, zc = L / (a.ntx * a.nty);
    double nrm[2] = {0.0, 0.0};
    march3r<R, T, K, NW, SITE, ZB, NORM, XP>(a, tab, tw, tx, ty, zc * a.zchunk, min(a.nz, (zc + 1) * a.zchunk), e, nrm);
    if constexpr (NORM) {
        const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) nrm[c] += __shfl_xor(nrm[c], off, 64);
            if (lane == 0) red[2 * wv + c] = nrm[c];
        }
        __syncthreads();
        if (threadIdx.x < 2) {
            double s = 0.0;
            for (int v = 0; v < NW; ++v) s += red[2 * v + threadIdx.x];
            a.npart[2 * (size_t)blockIdx.x + threadIdx.x] = s;
        }
    }
}

// A built shape: steps per launch, rows per thread, waves, waves per SIMD that its
// registers allow, workgroups a CU holds at once (by LDS), and the measured time of
// one iteration (half-plane) of a workgroup that has a CU to itself; two on a CU
// take 1.45 times that each.
struct M3Shape {
    int T, K, NW, WPE, occ;
    double iter_us;
};

// Tile width: 56 complex64 cells keep every row's stores on whole 64-byte pieces (60
// of them measured 13% slower at 512^3, partial lines being written twice); the full
// 64 - 2T where that saves one of at most five tile columns.  60 complex128 cells are
// whole pieces too and serve wherever they save a column (512^3: 7.15 against 7.62 ms
// per two steps; with as many columns 56, whole lines, is ahead: 256^3 0.87 and 0.92).
template <typename R> inline int m3_width(int nx, int T) {
    const int full = sizeof(R) == 8 ? std::min(60, 64 - 2 * T) : 64 - 2 * T;
    const int nf = (nx + full - 1) / full, n56 = (nx + 55) / 56;
    return (sizeof(R) == 8 || n56 <= 5) && nf < n56 ? full : 56;
}

// The fastest of a unit's shapes for T steps.  A unit names the precision R, whether
// per-site records come in (kRec), and its shapes (kShapes).  A chunk of p planes
// takes 2 p + 4 T iterations, of which the filling ones evaluate few levels: together
// they cost about 2 (p + T).  Workgroups run in rounds of one or two per CU.  A
// one-step launch with zero values outside, whose lanes without a cell load nothing,
// fills sooner and takes less where a tile is partly empty, but no less than its bytes
// at 8 TB/s out of the caches and 4.3 from memory.  Measured / estimated: complex64
// 128^3 75 / 76 us, 300 x 1 x 300 33 / 39, with records 128^3 99 / 98, 63 x 100 x 30 18 / 16,
// complex128 128^3 122 / 142, 63 x 100 x 30 20 / 21, 4 x 64 x 512 41 / 51.
// The last pick for each (T, boundary) is kept per thread.  Periodic rows that divide
// 64 need no ring in x: built for the shapes of one row per thread and two steps,
// which such lattices take (two steps of 64^3 with and without, when added: complex64
// 17.1 and 21 us, complex128 21.7 and 28, with records 28 and 39).
template <class U> static const M3Pick &m3_pick(int T, bool zb, int nx, int ny, int nz) {
    struct Memo {
        int nx = -1, ny = -1, nz = -1;
        M3Pick pick;
    };
    static thread_local Memo memo[4][2];
    Memo &m = memo[T & 3][zb ? 1 : 0];
    if (m.nx == nx && m.ny == ny && m.nz == nz) return m.pick;
    M3Pick best;
    const int64_t cus = resident_per_round();
    for (int q = 0; q < (int)std::size(U::kShapes); ++q) {
        const M3Shape &sh = U::kShapes[q];
        if (sh.T != T) continue;
        M3Pick p;
        p.shape = q;
        p.K = sh.K;
        p.NW = sh.NW;
        p.xp = !zb && T == 2 && sh.K == 1 && 64 % nx == 0;
        p.tw = p.xp ? nx : m3_width<typename U::R>(nx, T);
        p.nty = (ny + sh.K * sh.NW - 2 * T - 1) / (sh.K * sh.NW - 2 * T);
        const int64_t tiles = (int64_t)((nx + p.tw - 1) / p.tw) * p.nty;
        const double full = (double)nx * ny / ((double)tiles * p.tw * (sh.K * sh.NW - 2 * T));
        const bool partly = T == 1 && zb;
        const double iter_us = sh.iter_us * (partly ? 0.4 + 0.72 * full : 1.0), filling = partly ? 0.3 : T;
        for (int occ = 1; occ <= sh.occ; ++occ) {
            const int64_t per = cus * occ, cap = std::min<int64_t>(nz, 8 * ((per + tiles - 1) / tiles));
            for (int64_t c = 1; c <= cap; ++c) {
                p.nzc = (int)c;
                p.us = 4.0 + (double)((tiles * c + per - 1) / per) * 2.0 * ((double)((nz + c - 1) / c) + filling) *
                                 iter_us * (occ == 1 ? 1.0 : 1.45);
                if (best.shape < 0 || p.us < best.us) best = p;
            }
        }
    }
    if (T == 1 && zb) {
        const double bytes = (double)nx * ny * nz * 8.0 * sizeof(typename U::R) * (!U::kRec ? 4.0 : sizeof(typename U::R) == 4 ? 6.0 : 5.0);
        best.us = std::max(best.us, 4.0 + bytes / (bytes > 2e8 ? 4.3e6 : 8e6));
    }
    m.nx = nx;
    m.ny = ny;
    m.nz = nz;
    m.pick = best;
    return m.pick;
}

// REC: with per-site records, else with V(z) tables.
template <typename R, int T, int K, int NW, int WPE, bool REC>
hipError_t m3_launch(FusedArgs<R> a, const M3Pick &pick, bool zb, hipStream_t s, int *nblocks_out) {
    const int tw = pick.tw;
    a.ntx = (a.nx + tw - 1) / tw;
    a.nty = pick.nty;
    a.zchunk = (a.nz + pick.nzc - 1) / pick.nzc;
    a.nzc = (a.nz + a.zchunk - 1) / a.zchunk;
    const int64_t nblk = (int64_t)a.ntx * a.nty * a.nzc;
    if (nblk > 0x7fffffff) return hipErrorInvalidValue;
    if (nblocks_out) *nblocks_out = (int)nblk;
    const bool norm = a.npart != nullptr;
    if (norm && (nblk > a.npart_cap || a.rev || T > 2)) return hipErrorInvalidValue;
    const dim3 g((unsigned)nblk), b(NW * 64);
    // one step of a periodic complex128 lattice runs on the LDS march's kernel
    constexpr bool PERIODIC = T > 1 || sizeof(R) == 4;
#define M3(SITE, ZB, NORM)                                                                                          \
    do {                                                                                                            \
        constexpr bool XP = !ZB && T == 2 && K == 1;                                                                \
        if constexpr (!ZB && !PERIODIC)                                                                             \
            return hipErrorInvalidValue;                                                                            \
        else if (XP && pick.xp)                                                                                     \
            hipLaunchKernelGGL((k3_march3r<R, T, K, NW, WPE, SITE, ZB, NORM, XP>), g, b, 0, s, a, a.tab, tw);       \
        else                                                                                                        \
            hipLaunchKernelGGL((k3_march3r<R, T, K, NW, WPE, SITE, ZB, NORM, false>), g, b, 0, s, a, a.tab, tw);    \
    } while (0)
    if constexpr (T > 2) {
        if (zb) M3(0, true, false);
        else M3(0, false, false);
    } else if constexpr (!REC) {
        if (norm && zb) M3(0, true, true);
        else if (norm) M3(0, false, true);
        else if (zb) M3(0, true, false);
        else M3(0, false, false);
    } else {
        if (norm && zb) M3(1, true, true);
        else if (norm) M3(1, false, true);
        else if (a.rev && zb) M3(2, true, false);
        else if (a.rev) M3(2, false, false);
        else if (zb) M3(1, true, false);
        else M3(1, false, false);
    }
#undef M3
    return hipGetLastError();
}

// The launch of a pick among a unit's shapes.
template <class U, int I = 0>
hipError_t m3_run(const FusedArgs<typename U::R> &a, const M3Pick &p, bool zb, hipStream_t s, int *nblocks_out) {
    if constexpr (I < (int)std::size(U::kShapes)) {
        constexpr M3Shape S = U::kShapes[I];
        if (p.shape == I)
            return m3_launch<typename U::R, S.T, S.K, S.NW, S.WPE, U::kRec>(a, p, zb, s, nblocks_out);
        return m3_run<U, I + 1>(a, p, zb, s, nblocks_out);
    }
    return hipErrorInvalidValue;
}

// What a unit's source file defines.
#define M3_UNIT(U)                                                                                                  \
    template <> const M3Pick &march3r_pick_of<U::R, U::kRec>(int steps, bool zb, int nx, int ny, int nz) {          \
        return m3_pick<U>(steps, zb, nx, ny, nz);                                                                   \
    }                                                                                                               \
    template <>                                                                                                     \
    hipError_t launch_march3r_of<U::R, U::kRec>(const FusedArgs<U::R> &a, int steps, bool zb, hipStream_t s,        \
                                                int *nblocks_out) {                                                 \
        return m3_run<U>(a, m3_pick<U>(steps, zb, a.nx, a.ny, a.nz), zb, s, nblocks_out);                           \
    }

}  // namespace dirac
