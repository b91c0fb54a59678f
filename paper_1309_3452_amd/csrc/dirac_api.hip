// C ABI of the library: context, validation, coefficient tables, dispatch of
// the single-lattice kernels.  The batched entry points live in batch.hip.
#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <string>
#include <vector>

#include "../../include/dirac.h"
#include "adjmarch.h"
#include "cayley.h"
#include "ctx.h"
#include "gauge.h"
#include "internal.h"
#include "march3r_plan.h"
#include "tile2_plan.h"

using namespace dirac;

// ---------------------------------------------------------------------------
// helpers
// ---------------------------------------------------------------------------
namespace {

int fail(dirac_ctx *c, int code, const char *fmt, ...) __attribute__((format(printf, 3, 4)));
int fail(dirac_ctx *c, int code, const char *fmt, ...) {
    if (c) {
        char buf[512];
        va_list ap;
        va_start(ap, fmt);
        vsnprintf(buf, sizeof buf, fmt, ap);
        va_end(ap);
        c->err = buf;
    }
    return code;
}

#define HIPCHK(ctx, expr)                                                                         \
    do {                                                                                          \
        hipError_t e_ = (expr);                                                                   \
        if (e_ != hipSuccess)                                                                     \
            return fail((ctx), DIRAC_E_HIP, "%s: %s (%s:%d)", #expr, hipGetErrorString(e_), __FILE__, \
                        __LINE__);                                                                \
    } while (0)

bool finite_pos(double v) { return isfinite(v) && v > 0.0; }

size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

// Planes of the V(z) tables and per-site fields: the interior plus, in z-slab
// mode, the halo planes on both sides.
int64_t planes_of(const dirac_ctx *c) { return c->nz + 2 * c->zh; }

size_t array_bytes(const dirac_ctx *c) {
    return (size_t)c->nx * (size_t)c->ny * (size_t)planes_of(c) * (c->dtype == DIRAC_C64 ? 8u : 16u);
}

// Two arrays of that many bytes overlap.
bool ranges_meet(const void *a, const void *b, size_t bytes) {
    const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
    return x < y + bytes && y < x + bytes;
}

// theta of class q (A, B, C, D) at plane k: (dt/2)(+-m + V at the class's z).
double theta_of(const dirac_ctx *c, int q, int64_t k) {
    double h = 0.5 * c->dt;
    double v = 0.0;
    if (!c->v_int.empty()) v = (q == 0 || q == 3) ? c->v_int[k] : c->v_half[k];
    double sgn = (q < 2) ? 1.0 : -1.0;
    return h * (sgn * c->m + v);
}
// Im theta of class q at plane k: (dt/2) Im V at the class's z (m is real).
double theta_im_of(const dirac_ctx *c, int q, int64_t k) {
    if (c->w_int.empty()) return 0.0;
    return 0.5 * c->dt * ((q == 0 || q == 3) ? c->w_int[k] : c->w_half[k]);
}

template <typename R> size_t tab_bytes(const dirac_ctx *c) { return (size_t)4 * planes_of(c) * 4 * sizeof(R); }

size_t tab_bytes_of(const dirac_ctx *c) {
    return c->dtype == DIRAC_C64 ? tab_bytes<float>(c) : tab_bytes<double>(c);
}

// scratch layout
// Per-workgroup partials of the in-step functional (two doubles each): every
// z-march launch has at most nz chunks per tile column, and its tiles are at
// least 32 x 4 or 16 x 16 cells, so the area is sized for the larger tile
// count of the two and an in-step reduction is never refused for lack of
// slots.  The standalone reductions use kReduceBlocks x kObsVals doubles of the
// same area.
size_t step_partials(const dirac_ctx *c) {
    const size_t t1 = (size_t)((c->nx + 31) / 32) * (size_t)((c->ny + 3) / 4);
    const size_t t2 = (size_t)((c->nx + 15) / 16) * (size_t)((c->ny + 15) / 16);
    return (t1 > t2 ? t1 : t2) * (size_t)c->nz;
}
size_t partial_doubles(const dirac_ctx *c) {
    const size_t red = (size_t)kReduceBlocks * kObsVals, stp = 2 * step_partials(c);
    return red > stp ? red : stp;
}
size_t off_partial(const dirac_ctx *) { return 0; }
size_t off_result(const dirac_ctx *c) { return align256(partial_doubles(c) * sizeof(double)); }
size_t off_tab(const dirac_ctx *c) { return off_result(c) + 256; }
size_t off_gpart(const dirac_ctx *c) { return off_tab(c) + 2 * align256(tab_bytes_of(c)); }
size_t scratch_need(const dirac_ctx *c) {
    size_t g = 0;
    if (c->ndim == 3) g = (size_t)adj_tiles3((int)c->nx, (int)c->ny) * c->nz * 2 * sizeof(double);
    return off_gpart(c) + align256(g);
}

char *scratch_at(const dirac_ctx *c, size_t off) { return (char *)c->scratch + off; }

int upload_tables(dirac_ctx *c, hipStream_t s) {
    if (!c->tab_dirty) return DIRAC_OK;
    if (!c->scratch) return fail(c, DIRAC_E_STATE, "scratch must be bound before stepping");
    const int64_t nz = planes_of(c);
    if (c->dtype == DIRAC_C128) {
        c->tab_host64.assign((size_t)2 * 4 * nz * 4, 0.0);
        for (int dir = 0; dir < 2; ++dir)
            for (int q = 0; q < 4; ++q)
                for (int64_t k = 0; k < nz; ++k) {
                    double th = theta_of(c, q, k), thi = theta_im_of(c, q, k);
                    cayley64c(dir == 0 ? th : -th, dir == 0 ? thi : -thi,
                              &c->tab_host64[(((size_t)dir * 4 + q) * nz + k) * 4]);
                }
        size_t half = tab_bytes<double>(c);
        HIPCHK(c, hipMemcpyAsync(scratch_at(c, off_tab(c)), c->tab_host64.data(), half, hipMemcpyHostToDevice, s));
        HIPCHK(c, hipMemcpyAsync(scratch_at(c, off_tab(c) + align256(half)), c->tab_host64.data() + 4 * nz * 4,
                                 half, hipMemcpyHostToDevice, s));
    } else {
        // The unit-modulus search takes the host 1 us an entry (256 planes: 2.0 ms of a
        // first step) and the device 20 whatever their number, twice.  So up to six planes
        // (2D: one) the host forms the entries; beyond, theta goes up in their place and
        // becomes the entry there.  set_potential and a step, host / device: one plane 56 /
        // 97 us, four 80 / 99, eight 110 / 99.
        const bool on_host = nz <= 6;
        c->tab_host64.assign((size_t)2 * 4 * nz * 2, 0.0);
        for (int dir = 0; dir < 2; ++dir)
            for (int q = 0; q < 4; ++q)
                for (int64_t k = 0; k < nz; ++k) {
                    const double sg = dir == 0 ? 1.0 : -1.0;
                    const double th[2] = {sg * theta_of(c, q, k), sg * theta_im_of(c, q, k)};
                    double *e = &c->tab_host64[(((size_t)dir * 4 + q) * nz + k) * 2];
                    float entry[4];
                    if (on_host) cayley32c(th[0], th[1], entry);
                    memcpy(e, on_host ? (const void *)entry : (const void *)th, 16);
                }
        const size_t half = tab_bytes<float>(c);
        for (int dir = 0; dir < 2; ++dir) {
            void *t = scratch_at(c, off_tab(c) + dir * align256(half));
            HIPCHK(c, hipMemcpyAsync(t, c->tab_host64.data() + (size_t)dir * 4 * nz * 2, half, hipMemcpyHostToDevice, s));
            if (!on_host) HIPCHK(c, launch_table32(t, 4 * nz, s));
        }
    }
    // the host staging vectors stay alive in the context until the next upload
    HIPCHK(c, hipStreamSynchronize(s));
    c->tab_dirty = false;
    return DIRAC_OK;
}

template <typename R> HalfArgs<R> half_args(dirac_ctx *c, bool reverse) {
    HalfArgs<R> a;
    memset(&a, 0, sizeof a);
    int narr = c->ndim == 3 ? 8 : 4;
    for (int q = 0; q < narr; ++q) {
        a.f[q] = c->buf[c->cur][q];
        a.th[q] = c->site_mode ? (const R *)c->theta[q] : nullptr;
    }
    size_t half = align256(tab_bytes<R>(c));
    a.tab = c->site_mode ? nullptr : (const R *)scratch_at(c, off_tab(c) + (reverse ? half : 0));
    R sg = reverse ? (R)-1 : (R)1;
    a.rx = sg * (R)c->rx;
    a.ry = sg * (R)c->ry;
    a.rz = sg * (R)c->rz;
    a.tsgn = sg;
    a.nx = (int)c->nx;
    a.ny = (int)c->ny;
    a.nz = (int)c->nz;
    a.zbc = c->zbc ? 1 : 0;
    return a;
}

template <typename R> FusedArgs<R> fused_args(dirac_ctx *c) {
    FusedArgs<R> a;
    memset(&a, 0, sizeof a);
    int narr = c->ndim == 3 ? 8 : 4;
    for (int q = 0; q < narr; ++q) {
        a.in[q] = c->buf[c->cur][q];
        a.out[q] = c->buf[1 - c->cur][q];
        a.th[q] = c->site_mode ? (const R *)c->theta[q] : nullptr;
    }
    a.tab = c->site_mode ? nullptr : (const R *)scratch_at(c, off_tab(c));
    a.rx = (R)c->rx;
    a.ry = (R)c->ry;
    a.rz = (R)c->rz;
    a.nx = (int)c->nx;
    a.ny = (int)c->ny;
    a.nz = (int)c->nz;
    a.zchunk = c->zchunk;
    a.zh = c->zh;
    return a;
}

int kernel_choice(const dirac_ctx *c) {
    // the fused kernels address a plane with 32-bit byte offsets
    const uint64_t plane_bytes = (uint64_t)c->nx * (uint64_t)c->ny * (c->dtype == DIRAC_C64 ? 8u : 16u);
    if (c->zh) {
        // z-slab mode: the two-step march where it applies (the two halo planes
        // serve two steps), else the one-step march; never the split kernels
        if (c->kernel != DIRAC_KERNEL_FUSED && plane_bytes < (1ull << 32) &&
            fused3x2_supported((int)c->nx, c->dtype == DIRAC_C64, c->site_mode))
            return DIRAC_KERNEL_FUSED2;
        return DIRAC_KERNEL_FUSED;
    }
    if (c->kernel == DIRAC_KERNEL_SPLIT) return DIRAC_KERNEL_SPLIT;
    // zero values outside the lattice: the split kernels (in place)
    if (c->zbc) return DIRAC_KERNEL_SPLIT;
    // links: the link marches (one step per launch)
    if (c->links_on) return DIRAC_KERNEL_FUSED;
    if (plane_bytes >= (1ull << 32)) return DIRAC_KERNEL_SPLIT;
    if (c->kernel == DIRAC_KERNEL_FUSED) return DIRAC_KERNEL_FUSED;
    if (c->ndim == 3 && fused3x2_supported((int)c->nx, c->dtype == DIRAC_C64, c->site_mode))
        return DIRAC_KERNEL_FUSED2;
    // (2+1)D: a two-step pass recomputes a six-row pipeline per chunk, so small
    // lattices (under 2^18 cells, cache-resident) keep the one-step march, which
    // spreads them over more workgroups; an explicit FUSED2 request is honoured
    if (c->ndim == 2 && fused2x2_supported((int)c->nx, c->dtype == DIRAC_C64) &&
        (c->kernel == DIRAC_KERNEL_FUSED2 || c->nx * c->ny >= (int64_t)1 << 18))
        return DIRAC_KERNEL_FUSED2;
    return DIRAC_KERNEL_FUSED;
}

// Buffer-set flips of n steps by kernel_choice's kernel: they decide which set
// ends up with the state.
int64_t flips_of(const dirac_ctx *c, int64_t n) {
    const int kc = kernel_choice(c);
    return kc == DIRAC_KERNEL_SPLIT ? 0 : kc == DIRAC_KERNEL_FUSED2 ? n / 2 + (n & 1) : n;
}

// The two buffer sets share memory: only the in-place kernels can take that.
bool sets_shared(const dirac_ctx *c) {
    const int narr = c->ndim == 3 ? 8 : 4;
    const size_t bytes = array_bytes(c);
    for (int q = 0; q < narr; ++q)
        for (int p = 0; p < narr; ++p)
            if (ranges_meet(c->buf[0][q], c->buf[1][p], bytes)) return true;
    return false;
}

// (2+1)D with the kernel and its knobs left to the library: several steps per
// pass on register tiles (tile2.hip).
bool tile2_applies(const dirac_ctx *c) {
    return c->ndim == 2 && c->kernel == DIRAC_KERNEL_AUTO && c->zchunk == 0 && !sets_shared(c);
}

// The register marches address a plane, and a V(z) table of four classes, with
// 32-bit byte offsets (a complex128 table reaches 4 GiB at 2^25 planes).
bool offsets_fit(const dirac_ctx *c) {
    const uint64_t plane = (uint64_t)c->nx * (uint64_t)c->ny * (c->dtype == DIRAC_C64 ? 8u : 16u);
    return plane < (1ull << 32) && (c->site_mode || tab_bytes_of(c) < (1ull << 32));
}

bool narrow_on_lds(const dirac_ctx *c) {
    if (c->dtype != DIRAC_C128 || c->site_mode || c->zbc || c->nx > 16) return false;
    const int nx = (int)c->nx, ny = (int)c->ny, nz = (int)c->nz;
    return march_lds_wins_narrow(march3r_us<double>(2, false, false, nx, ny, nz), nx, ny, nz);
}

// (3+1)D likewise: the register march (march3r.h) where it is the fastest kernel.
// Per launch of two steps, next to the LDS march (one-step one for an odd
// complex64 width, split kernels with zero values outside): complex128 256^3
// 0.87 against 0.99 ms, 64^3 21 against 37 us, with records 200 x 168 x 152 0.41
// against 0.69 ms; complex64 191 x 151 x 127 0.14 against 0.30, zero values outside
// 224 x 192 x 256 0.29 against 0.96.  For complex64 of even width the two are
// close and the tiles' fit decides (tables: 32^3 9 against 21 us, 64^3 15 / 26,
// 96^3 34 / 50, 128^3 88 / 79, 160^3 129 / 142, 256^3 545 / 447; records: 96^3 50 /
// 79, 128^3 125 / 111, 200 x 168 x 152 251 / 342, 256^3 789 / 756): the estimates of
// both, the register march's less 5%.
bool march3_applies(const dirac_ctx *c) {
    if (c->ndim != 3 || c->kernel != DIRAC_KERNEL_AUTO || c->tile_y != 0 || c->zchunk != 0 || c->links_on || c->zh)
        return false;
    if (!offsets_fit(c) || narrow_on_lds(c)) return false;
    if (!c->zbc && c->dtype == DIRAC_C64 && c->nx % 2 == 0) {
        const int nx = (int)c->nx, ny = (int)c->ny, nz = (int)c->nz;
        if (march3r_us<float>(2, c->site_mode, false, nx, ny, nz) > 0.95 * march_lds_us(c->site_mode, nx, ny, nz)) return false;
    }
    return !sets_shared(c);
}

// Two steps of a z-slab in one launch: complex128 slabs take the register march too,
// whose two-step reach is the slab's two halo planes (512 x 512 x 64: 0.90 against 1.08
// ms, with records 1.45 against 1.91).
bool slab_on_march3(const dirac_ctx *c) {
    return c->ndim == 3 && c->zh && c->dtype == DIRAC_C128 && c->kernel == DIRAC_KERNEL_AUTO && c->zchunk == 0 &&
           !narrow_on_lds(c);
}

// z-slab mode: the most steps one call may advance between halo refills
int halo_steps(const dirac_ctx *c) { return kernel_choice(c) == DIRAC_KERNEL_FUSED2 ? 2 : 1; }

int slab_step_check(dirac_ctx *c, int64_t n) {
    if (c->zh && n > halo_steps(c))
        return fail(c, DIRAC_E_ARG, halo_steps(c) == 2 ? "z-slab mode: at most 2 steps per call, halos refilled between calls"
                                                       : "z-slab mode: 1 step per call, halos refilled between calls");
    return DIRAC_OK;
}

LinkPtrs link_ptrs(const dirac_ctx *c) {
    LinkPtrs L;
    for (int q = 0; q < 24; ++q) L.u[q] = c->links[q];
    return L;
}

// n steps as `splits` in-place steps of the split kernels (zero values outside only),
// then launches of three, two and one steps.
struct March3Plan {
    int64_t splits = 0, threes = 0, twos = 0, ones = 0;
    int64_t launches() const { return threes + twos + ones; }
};

// Estimated microseconds of a (3+1)D step on the split kernels, and of the functional
// as a reduction over the state.  A thread costs 22 ps, with a cell or without, a cell
// at least 33 (complex64) or 64 ps, half as much again where rows start off the
// 64-byte pieces (not in complex128 up to 30 MB) and 1.42 times from memory rather than
// the caches; all 1.18 times with records; two launches take 7.8 (9.0) at least.
// Measured / estimated, zero values outside: complex64 4 x 64 x 512 49 / 50, 33 x 40 x 50
// 8.7 / 7.8, 128^3 66 / 73, 129^3 109 / 110, 200 x 168 x 152 224 / 243, complex128
// 63 x 100 x 30 14 / 16, 128^3 124 / 138, 1 x 300 x 300 103 / 130, with records 125 / 153.
double split3_us(const dirac_ctx *c) {
    const bool fp32 = c->dtype == DIRAC_C64;
    const double cells = (double)c->nx * (double)c->ny * (double)c->nz, bytes = cells * (fp32 ? 64.0 : 128.0);
    const double threads = (double)((c->nx + 63) / 64 * 64) * (double)((c->ny + 3) / 4 * 4) * (double)c->nz;
    double ps = fp32 ? 33.0 : 64.0;
    if (c->nx * (fp32 ? 8 : 16) % 64 != 0 && (fp32 || bytes > 3e7)) ps *= 1.5;
    if (bytes > 3e8) ps *= 1.42;
    const double us = 1e-6 * std::max(22.0 * threads, ps * cells) * (c->site_mode ? 1.18 : 1.0);
    return std::max(fp32 ? 7.8 : 9.0, 3.5 + us);
}
double norm3_us(const dirac_ctx *c) {
    return 30.0 + 20e-6 * (double)((c->nx + 63) / 64 * 64) * (double)((c->ny + 3) / 4 * 4) * (double)c->nz;
}

// A plan's one-step launches take the LDS march's one-step kernel where its rows are
// whole (257^3 complex128: 0.84 against 0.97 ms), and in a single row of them (301 x 1 x
// 300 complex64 26 against 29 us; with records level).
bool ones_on_fused(const dirac_ctx *c) {
    return !c->zbc && (c->dtype == DIRAC_C128 || c->nx % 2 == 0 || (c->ny == 1 && !c->site_mode));
}

// The split of n with the least estimated time whose launches have the parity of
// `flips`; with sum_last its last launch has at most two steps (it also sums the
// functional, for a fifth of its time more).  With zero values outside in-place steps
// may come in too: two of them in place of two one-step launches are as fast or faster
// on boxes of up to about 128^3 (two steps of 128^3 complex64 131 against 151 us, 63 x 100
// x 30 complex128 28 against 40, 200 x 168 x 152 complex64 448 against 310).  False if
// there is no plan or in-place steps alone are the fastest (n = 1 with an even number
// of flips; n = 0).
template <typename R> bool plan_march3(const dirac_ctx *c, int64_t n, int64_t flips, bool sum_last, March3Plan *out) {
    const int most = march3r_most(sizeof(R) == 4, c->site_mode);
    double us[4] = {};
    const int nx = (int)c->nx, ny = (int)c->ny, nz = (int)c->nz;
    for (int t = 1; t <= most; ++t)
        us[t] = t == 1 && ones_on_fused(c) ? fused3_us(sizeof(R) == 4, c->site_mode, nx, ny, nz)
                                           : march3r_us<R>(t, c->site_mode, c->zbc, nx, ny, nz);
    const double split = c->zbc ? split3_us(c) : 0.0;
    bool found = false;
    double best = c->zbc ? (double)n * split + (sum_last ? norm3_us(c) : 0.0) : 1e300;
    for (int64_t splits = 0; splits <= (c->zbc ? 3 : 0); ++splits) {
        const int64_t m = n - splits;
        const int64_t lo = (m + most - 1) / most, hi = m / 2 + 3 < m ? m / 2 + 3 : m;
        for (int64_t p = lo; p <= hi; ++p) {
            if (p < 1 || ((p ^ flips) & 1)) continue;
            March3Plan q;
            q.splits = splits;
            if (2 * p >= m) {
                q.twos = m - p;
                q.ones = 2 * p - m;
            } else {
                q.threes = m - 2 * p;
                q.twos = 3 * p - m;
            }
            if (sum_last && q.twos + q.ones == 0) continue;
            const double t = (double)splits * split + (double)q.threes * us[3] + (double)q.twos * us[2] +
                             (double)q.ones * us[1] + (sum_last ? 0.2 * us[q.ones ? 1 : 2] : 0.0);
            if (t < best) {
                found = true;
                best = t;
                *out = q;
            }
        }
    }
    return found;
}

// Estimated microseconds of n (2+1)D steps on the kernels before the register tiles:
// in place on the split kernels (zero values outside, reversed steps) or, up to 8 rows,
// by row marches.  Split: a thread costs 10.5 ps, a cell at least 20 (complex64) or 36
// ps, 23 and 39 from memory, 0.85 of that without records.  Marches: a cell of one step
// 18 ps in complex64 without a potential, the others as in the table; two steps in one
// launch 1.35 times one.  Measured / estimated per step: in place 100000 x 5 complex64 per
// site 11 / 12 us, complex128 19 / 20, 400000 x 1 complex128 13 / 19, 8 x 100000 73 / 69; marches
// 400000 x 1 complex64 12 / 12, 400000 x 4 33 / 34, complex128 per site 75 / 72, with links
// 99 / 101.
double before_tiles_us(const dirac_ctx *c, int64_t n, bool in_place) {
    const bool fp32 = c->dtype == DIRAC_C64;
    const double cells = (double)c->nx * (double)c->ny;
    if (in_place) {
        const double threads = (double)((c->nx + 63) / 64 * 64) * (double)((c->ny + 3) / 4 * 4);
        const bool far = cells * (fp32 ? 32.0 : 64.0) > 2e8;
        const double ps = (fp32 ? (far ? 23.0 : 20.0) : (far ? 39.0 : 36.0)) * (c->site_mode ? 1.0 : 0.85);
        return (double)n * std::max(6.9, 2.0 + 1e-6 * std::max(10.5 * threads, ps * cells));
    }
    if (c->ny > 8) return 1e300;
    constexpr double ps[2][4] = {{36.0, 42.0, 60.0, 66.0}, {18.0, 22.0, 30.0, 34.0}};
    const double one = std::max(6.4, 5.0 + 1e-6 * ps[fp32 ? 1 : 0][tile2_kind(c->site_mode, c->links_on)] * cells);
    if (kernel_choice(c) != DIRAC_KERNEL_FUSED2) return (double)n * one;
    return (double)(n / 2) * 1.35 * one + (double)(n & 1) * one;
}

// Whether that many passes of register tiles are the faster way.  Up to a round and a
// half of tiles they are.  Beyond, a few long rows leave a region mostly empty
// (one step of 400000 x 1 complex128 per site 76 against 21 us, of 400000 x 4 95 against
// 75, of 400000 x 12 183 against 179; two in place of 100000 x 2 with zero values
// outside 38 against 16), and so do narrow planes of complex128 records in place
// (8 x 100000, two steps 171 against 145).
bool tiles_win(const dirac_ctx *c, int64_t n, int64_t passes, bool in_place) {
    if (2 * tile2_tiles(0, 1, c->nx, c->ny) <= 3 * (int64_t)resident_per_round()) return true;
    return tile2_total_us(n, passes, c->nx, c->ny, c->dtype == DIRAC_C64, tile2_kind(c->site_mode, c->links_on)) <=
           before_tiles_us(c, n, in_place);
}

// What a call launches, decided here for the call itself and for dirac_route.
enum class Op { step, reverse, step_norm };
enum class Way { split, fused, fused2, tile2, march3 };
struct Route {
    Way way = Way::split;
    int64_t passes = 0;      // tile2
    March3Plan plan;         // march3; of reversed steps those between the two half-steps
};

Way way_of(int kc) {
    return kc == DIRAC_KERNEL_FUSED2 ? Way::fused2 : kc == DIRAC_KERNEL_FUSED ? Way::fused : Way::split;
}

template <typename R> Route route_of(const dirac_ctx *c, int64_t n, Op op) {
    Route r;
    const int kc = kernel_choice(c);
    // the buffer sets end up as kernel_choice's kernel would leave them; step_norm by
    // it makes its last launch (two steps or one) apart
    const int64_t flips = op == Op::reverse || n == 0 ? 0
                          : op == Op::step            ? flips_of(c, n)
                          : c->ndim == 3 && kc == DIRAC_KERNEL_FUSED2 && n >= 2 ? flips_of(c, n - 2) + 1
                                                                                : flips_of(c, n - 1) + flips_of(c, 1);
    if (tile2_applies(c) && !(op == Op::reverse && c->links_on)) {
        r.passes = tile2_passes(n, (int)(flips & 1), 1, &c->nx, &c->ny, sizeof(R) == 4,
                                tile2_kind(c->site_mode, c->links_on));
        if (r.passes > 0 && tiles_win(c, n, r.passes, c->zbc || op == Op::reverse)) {
            r.way = Way::tile2;
            return r;
        }
    }
    if (op == Op::reverse) {
        const bool march = march3_applies(c);
        // 3D lattices whose forward steps take a march kernel reverse on it too
        const bool old_march = c->ndim == 3 && !c->links_on && !c->zh && kc != DIRAC_KERNEL_SPLIT;
        if ((old_march || n > 2) && march && (n == 1 || plan_march3<R>(c, n - 1, flips_of(c, n - 1), false, &r.plan)))
            r.way = Way::march3;
        else
            r.way = old_march ? way_of(kc) : Way::split;
        return r;
    }
    r.way = march3_applies(c) && plan_march3<R>(c, n, flips, op == Op::step_norm, &r.plan) ? Way::march3 : way_of(kc);
    return r;
}

// The forward march kernels run the reversed sequence: with r -> -r, the
// reversed coefficient tables (theta -> -theta) and per-site records read with
// theta -> -theta they apply H1' then H2', the two half-steps solved backwards
// (H1' undoes ss1, ss2; H2' undoes ss3, ss4).  n reversed steps are
// (H1' H2')^n = H1' (H2' H1')^(n-1) H2': one split H2', n - 1 march steps, one
// split H1'.
template <typename R> FusedArgs<R> fused_args_rev(dirac_ctx *c) {
    FusedArgs<R> a = fused_args<R>(c);
    a.rx = -a.rx;
    a.ry = -a.ry;
    a.rz = -a.rz;
    if (!c->site_mode) a.tab = (const R *)scratch_at(c, off_tab(c) + align256(tab_bytes<R>(c)));
    a.rev = 1;
    return a;
}

// The launches of a plan, forward or of the reversed sequence; with npart the
// last one sums the functional and *nblocks receives its workgroups.
template <typename R>
int run_march3(dirac_ctx *c, const March3Plan &plan, bool rev, hipStream_t s, double *npart, int npart_cap, int *nblocks) {
    for (int64_t t = 0; t < plan.splits; ++t)
        for (int which = 0; which < 2; ++which)        // A,B then C,D; reversed steps in between are H1' H2' too
            HIPCHK(c, launch_half3<R>(half_args<R>(c, rev), which, c->site_mode, s));
    const int64_t p = plan.launches();
    for (int64_t t = 0; t < p; ++t) {
        FusedArgs<R> a = rev ? fused_args_rev<R>(c) : fused_args<R>(c);
        if (npart && t + 1 == p) {
            a.npart = npart;
            a.npart_cap = npart_cap;
        }
        const int steps = t < plan.threes ? 3 : t < plan.threes + plan.twos ? 2 : 1;
        if (steps == 1 && ones_on_fused(c))
            HIPCHK(c, launch_fused3<R>(a, c->site_mode, 0, s, nblocks));
        else
            HIPCHK(c, launch_march3r<R>(a, steps, c->site_mode, c->zbc, s, nblocks));
        c->cur = 1 - c->cur;
    }
    return DIRAC_OK;
}

template <typename R> int run_reverse_march(dirac_ctx *c, int64_t n, const Route &r, hipStream_t s) {
    if (n <= 0) return DIRAC_OK;
    const bool site = c->site_mode;
    HIPCHK(c, launch_half3<R>(half_args<R>(c, true), 1, site, s));      // H2'
    if (r.way == Way::march3) {
        const int rc = run_march3<R>(c, r.plan, true, s, nullptr, 0, nullptr);
        if (rc) return rc;
        HIPCHK(c, launch_half3<R>(half_args<R>(c, true), 0, site, s));  // H1'
        return DIRAC_OK;
    }
    int64_t t = 1;
    if (r.way == Way::fused2) {
        for (; t + 2 <= n; t += 2) {
            HIPCHK(c, launch_fused3x2<R>(fused_args_rev<R>(c), site, s));
            c->cur = 1 - c->cur;
        }
    }
    for (; t < n; ++t) {
        HIPCHK(c, launch_fused3<R>(fused_args_rev<R>(c), site, c->tile_y, s));
        c->cur = 1 - c->cur;
    }
    HIPCHK(c, launch_half3<R>(half_args<R>(c, true), 0, site, s));      // H1'
    return DIRAC_OK;
}

// n steps on register tiles in that many passes.
template <typename R> int run_tile2(dirac_ctx *c, int64_t n, bool reverse, int64_t passes, hipStream_t s) {
    for (int64_t p = 0; p < passes; ++p) {
        const FusedArgs<R> a = reverse ? fused_args_rev<R>(c) : fused_args<R>(c);
        const int steps = (int)(n / passes + (p < n % passes));
        HIPCHK(c, c->links_on ? launch_tile2_links<R>(a, link_ptrs(c), c->site_mode, steps, s)
                              : launch_tile2<R>(a, c->site_mode, c->zbc, steps, s));
        c->cur = 1 - c->cur;
    }
    return DIRAC_OK;
}

// Two steps of a (3+1)D lattice or z-slab in one launch.
template <typename R> hipError_t launch_two(const dirac_ctx *c, const FusedArgs<R> &a, hipStream_t s, int *nblocks) {
    if (slab_on_march3(c)) return launch_march3r<R>(a, 2, c->site_mode, false, s, nblocks);
    return launch_fused3x2<R>(a, c->site_mode, s, nblocks);
}

template <typename R> int run_steps(dirac_ctx *c, int64_t n, bool reverse, hipStream_t s) {
    int rc = upload_tables(c, s);
    if (rc) return rc;
    const Route r = route_of<R>(c, n, reverse ? Op::reverse : Op::step);
    if (r.way == Way::tile2) return run_tile2<R>(c, n, reverse, r.passes, s);
    if (reverse && r.way != Way::split) return run_reverse_march<R>(c, n, r, s);
    if (r.way == Way::march3) return run_march3<R>(c, r.plan, false, s, nullptr, 0, nullptr);
    const bool site = c->site_mode;
    const bool fused = r.way != Way::split;
    int64_t t = 0;
    if (r.way == Way::fused2) {
        for (; t + 2 <= n; t += 2) {
            FusedArgs<R> a = fused_args<R>(c);
            if (c->ndim == 3) HIPCHK(c, launch_two<R>(c, a, s, nullptr));
            else HIPCHK(c, launch_fused2x2<R>(a, site, s));
            c->cur = 1 - c->cur;
        }
    }
    for (; t < n; ++t) {
        if (fused && c->links_on) {
            FusedArgs<R> a = fused_args<R>(c);
            if (c->ndim == 3) HIPCHK(c, launch_fused_links<R>(a, link_ptrs(c), site, s));
            else HIPCHK(c, launch_fused2_links<R>(a, link_ptrs(c), site, s));
            c->cur = 1 - c->cur;
        } else if (fused) {
            FusedArgs<R> a = fused_args<R>(c);
            if (c->ndim == 3) HIPCHK(c, launch_fused3<R>(a, site, c->tile_y, s));
            else HIPCHK(c, launch_fused2<R>(a, site, s));
            c->cur = 1 - c->cur;
        } else {
            HalfArgs<R> a = half_args<R>(c, reverse);
            int first = reverse ? 1 : 0;
            if (c->links_on) {
                const LinkPtrs L = link_ptrs(c);
                HIPCHK(c, launch_half_links<R>(a, L, c->ndim, first, site, s));
                HIPCHK(c, launch_half_links<R>(a, L, c->ndim, 1 - first, site, s));
            } else if (c->ndim == 3) {
                HIPCHK(c, launch_half3<R>(a, first, site, s));
                HIPCHK(c, launch_half3<R>(a, 1 - first, site, s));
            } else {
                HIPCHK(c, launch_half2<R>(a, first, site, s));
                HIPCHK(c, launch_half2<R>(a, 1 - first, site, s));
            }
        }
    }
    return DIRAC_OK;
}

// The launches of a route in their order: name, count and what tells their shape.
template <typename R> std::string route_text(const dirac_ctx *c, int64_t n, Op op) {
    const Route r = route_of<R>(c, n, op);
    const bool fp32 = sizeof(R) == 4;
    std::string t;
    auto add = [&t](int64_t count, const char *fmt, auto... v) {
        if (count < 1) return;
        char b[160];
        snprintf(b, sizeof b, fmt, v...);
        t += (t.empty() ? "" : "; ") + std::to_string((long long)count) + " x " + b;
    };
    const bool halves = op == Op::reverse && r.way != Way::split && r.way != Way::tile2 && n > 0;
    int64_t m = halves ? n - 1 : n;
    if (halves) add(1, "%s", "half");
    if (r.way == Way::tile2) {
        const int kind = tile2_kind(c->site_mode, c->links_on);
        for (const int64_t more : {(int64_t)1, (int64_t)0}) {
            const int steps = (int)(n / r.passes + more);
            double us = 0.0;
            const int64_t count = more ? n % r.passes : r.passes - n % r.passes;
            if (count)
                add(count, "tile2%s steps=%d rows=%d", c->links_on ? " links" : "", steps,
                    tile2_rows(tile2_best_shape(steps, 1, &c->nx, &c->ny, fp32, kind, &us)));
        }
    } else if (r.way == Way::march3) {
        add(r.plan.splits, "%s", "split");
        const int64_t counts[4] = {0, r.plan.ones, r.plan.twos, r.plan.threes};
        for (int T = 3; T > 0; --T) {
            if (counts[T] == 0) continue;
            if (T == 1 && ones_on_fused(c)) {
                add(counts[T], "%s", "fused");
                continue;
            }
            const M3Pick &p = march3r_pick<R>(T, c->site_mode, c->zbc, (int)c->nx, (int)c->ny, (int)c->nz);
            add(counts[T], "march3r steps=%d rows=%d waves=%d width=%d chunks=%d%s", T, p.K, p.NW, p.tw, p.nzc,
                p.xp ? " rotating" : "");
        }
    } else {
        if (r.way == Way::fused2) add(m / 2, "%s", slab_on_march3(c) ? "march3r steps=2" : "fused2");
        if (r.way == Way::fused2) m &= 1;
        add(m, "%s", r.way == Way::split ? "split" : c->links_on ? "fused links" : "fused");
    }
    if (halves) add(1, "%s", "half");
    return t;
}

template <typename R> ReduceArgs<R> reduce_args(dirac_ctx *c, double z0) {
    ReduceArgs<R> a;
    memset(&a, 0, sizeof a);
    int narr = c->ndim == 3 ? 8 : 4;
    for (int q = 0; q < narr; ++q) a.f[q] = c->buf[c->cur][q];
    a.rx = (R)c->rx;
    a.ry = (R)c->ry;
    a.rz = (R)c->rz;
    a.nx = (int)c->nx;
    a.ny = (int)c->ny;
    a.nz = (int)c->nz;
    a.z0 = z0;
    a.partial = (double *)scratch_at(c, off_partial(c));
    a.zh = c->zh;
    a.zbc = c->zbc ? 1 : 0;
    return a;
}

// Backward steps of the adjoint as one launch each, two at a time, given arrays to
// ping-pong with.
bool adjoint_on_march(const dirac_ctx *c, int64_t n) {
    if (c->ndim != 3 || c->site_mode || c->links_on || c->zh || c->zbc || !c->w_int.empty() || n < 2) return false;
    return offsets_fit(c) && !sets_shared(c) &&
           adj_march_wins(c->dtype == DIRAC_C64, (int)c->nx, (int)c->ny, (int)c->nz);
}

int check_ready(dirac_ctx *c, bool need_scratch) {
    if (!c) return DIRAC_E_ARG;
    if (c->is_batch) return fail(c, DIRAC_E_STATE, "batch context: use the dirac_batch_* calls");
    if (!c->bound) return fail(c, DIRAC_E_STATE, "no state bound (dirac_bind_state)");
    if (need_scratch && !c->scratch) return fail(c, DIRAC_E_STATE, "no scratch bound (dirac_bind_scratch)");
    return DIRAC_OK;
}

}  // namespace

// ---------------------------------------------------------------------------
// ABI
// ---------------------------------------------------------------------------
extern "C" {

const char *dirac_status_string(int status) {
    switch (status) {
    case DIRAC_OK: return "ok";
    case DIRAC_E_ARG: return "invalid argument";
    case DIRAC_E_SHAPE: return "invalid shape";
    case DIRAC_E_UNSTABLE: return "step above the stability bound";
    case DIRAC_E_NONFINITE: return "non-finite value";
    case DIRAC_E_HIP: return "HIP runtime error";
    case DIRAC_E_STATE: return "call out of order";
    default: return "unknown status";
    }
}

int dirac_create(dirac_ctx **out, int ndim, int64_t nx, int64_t ny, int64_t nz, int dtype, double dt, double dx,
                 double dy, double dz, unsigned flags) {
    if (!out) return DIRAC_E_ARG;
    *out = nullptr;
    if (ndim != 2 && ndim != 3) return DIRAC_E_ARG;
    if (dtype != DIRAC_C64 && dtype != DIRAC_C128) return DIRAC_E_ARG;
    if ((flags & ~(DIRAC_ALLOW_UNSTABLE | DIRAC_SLAB_Z | DIRAC_ZERO_BC)) != 0) return DIRAC_E_ARG;
    if ((flags & DIRAC_SLAB_Z) && ndim != 3) return DIRAC_E_ARG;
    if ((flags & DIRAC_SLAB_Z) && (flags & DIRAC_ZERO_BC)) return DIRAC_E_ARG;
    if (nx < 1 || ny < 1 || nz < 1) return DIRAC_E_SHAPE;
    if (ndim == 2 && nz != 1) return DIRAC_E_SHAPE;
    if (nx > (1 << 30) || ny > (1 << 30) || nz > (1 << 30)) return DIRAC_E_SHAPE;
    if ((double)nx * (double)ny * (double)nz >= 1099511627776.0) return DIRAC_E_SHAPE;
    if (!finite_pos(dt) || !finite_pos(dx) || !finite_pos(dy) || (ndim == 3 && !finite_pos(dz))) return DIRAC_E_ARG;
    double rx = dt / dx, ry = dt / dy, rz = ndim == 3 ? dt / dz : 0.0;
    double r2 = rx * rx + ry * ry + rz * rz;
    if (r2 > 1.0 + 1e-12 && !(flags & DIRAC_ALLOW_UNSTABLE)) return DIRAC_E_UNSTABLE;
    dirac_ctx *c = new (std::nothrow) dirac_ctx();
    if (!c) return DIRAC_E_ARG;
    c->ndim = ndim;
    c->nx = nx;
    c->ny = ny;
    c->nz = nz;
    c->dtype = dtype;
    c->dt = dt;
    c->rx = rx;
    c->ry = ry;
    c->rz = rz;
    c->flags = flags;
    c->zh = (flags & DIRAC_SLAB_Z) ? 2 : 0;
    c->zbc = (flags & DIRAC_ZERO_BC) != 0;
    *out = c;
    return DIRAC_OK;
}

void dirac_destroy(dirac_ctx *c) {
    if (!c) return;
    for (int p = 0; p < 2; ++p) {
        if (c->graph_exec[p]) (void)hipGraphExecDestroy(c->graph_exec[p]);
        if (c->graph[p]) (void)hipGraphDestroy(c->graph[p]);
    }
    delete c;
}

const char *dirac_last_error(const dirac_ctx *c) { return c ? c->err.c_str() : "null context"; }

int dirac_bind_state(dirac_ctx *c, void *const buf0[], void *const buf1[]) {
    if (!c || !buf0 || !buf1) return DIRAC_E_ARG;
    if (c->is_batch) return fail(c, DIRAC_E_STATE, "batch context: use dirac_batch_bind");
    int narr = c->ndim == 3 ? 8 : 4;
    for (int q = 0; q < narr; ++q)
        if (!buf0[q] || !buf1[q]) return fail(c, DIRAC_E_ARG, "null state array %d", q);
    for (int q = 0; q < 8; ++q) {
        c->buf[0][q] = q < narr ? buf0[q] : nullptr;
        c->buf[1][q] = q < narr ? buf1[q] : nullptr;
    }
    c->bound = true;
    c->cur = 0;
    return DIRAC_OK;
}

int dirac_current(const dirac_ctx *c, int *which) {
    if (!c || !which) return DIRAC_E_ARG;
    *which = c->cur;
    return DIRAC_OK;
}

int dirac_set_current(dirac_ctx *c, int which) {
    if (!c || (which != 0 && which != 1)) return DIRAC_E_ARG;
    c->cur = which;
    return DIRAC_OK;
}

int dirac_halo_steps(const dirac_ctx *c, int *steps) {
    if (!c || !steps) return DIRAC_E_ARG;
    *steps = (!c->is_batch && c->zh) ? halo_steps(c) : 0;
    return DIRAC_OK;
}

int dirac_scratch_bytes(const dirac_ctx *c, size_t *bytes) {
    if (!c || !bytes) return DIRAC_E_ARG;
    *bytes = c->is_batch ? c->batch_scratch_need : scratch_need(c);
    return DIRAC_OK;
}

int dirac_bind_scratch(dirac_ctx *c, void *dev, size_t bytes) {
    if (!c || !dev) return DIRAC_E_ARG;
    if (((uintptr_t)dev & 255) != 0) return fail(c, DIRAC_E_ARG, "scratch must be 256-byte aligned");
    size_t need = c->is_batch ? c->batch_scratch_need : scratch_need(c);
    if (bytes < need) return fail(c, DIRAC_E_SHAPE, "scratch too small: %zu < %zu bytes", bytes, need);
    c->scratch = dev;
    c->scratch_bytes = bytes;
    c->tab_dirty = true;
    return DIRAC_OK;
}

int dirac_set_potential_im_z(dirac_ctx *c, const double *w_int, const double *w_half, int64_t nz) {
    if (!c) return DIRAC_E_ARG;
    if (c->is_batch) return fail(c, DIRAC_E_STATE, "batch context");
    if (nz != planes_of(c))
        return fail(c, DIRAC_E_SHAPE, "nz %lld != lattice planes %lld", (long long)nz, (long long)planes_of(c));
    if ((w_int == nullptr) != (w_half == nullptr)) return fail(c, DIRAC_E_ARG, "w_int and w_half: both or neither");
    std::vector<double> wi, wh;
    if (w_int) {
        wi.assign(w_int, w_int + nz);
        wh.assign(w_half, w_half + nz);
        bool any = false;
        for (int64_t k = 0; k < nz; ++k) {
            if (!isfinite(wi[k]) || !isfinite(wh[k]))
                return fail(c, DIRAC_E_NONFINITE, "non-finite Im V at k=%lld", (long long)k);
            any = any || wi[k] != 0.0 || wh[k] != 0.0;
        }
        if (!any) {
            wi.clear();
            wh.clear();
        }
    }
    c->w_int.swap(wi);
    c->w_half.swap(wh);
    c->tab_dirty = true;
    return DIRAC_OK;
}

int dirac_set_mass_potential_z(dirac_ctx *c, double m, const double *v_int, const double *v_half, int64_t nz) {
    if (!c || !isfinite(m)) return DIRAC_E_ARG;
    if (c->is_batch) return fail(c, DIRAC_E_STATE, "batch context");
    if (nz != planes_of(c))
        return fail(c, DIRAC_E_SHAPE, "nz %lld != lattice planes %lld", (long long)nz, (long long)planes_of(c));
    if ((v_int == nullptr) != (v_half == nullptr)) return fail(c, DIRAC_E_ARG, "v_int and v_half: both or neither");
    if (v_int && c->ndim == 2) return fail(c, DIRAC_E_ARG, "2D: use dirac_theta_from_fields for V(x, y)");
    std::vector<double> vi, vh;
    if (v_int) {
        vi.assign(v_int, v_int + nz);
        vh.assign(v_half, v_half + nz);
        for (int64_t k = 0; k < nz; ++k)
            if (!isfinite(vi[k]) || !isfinite(vh[k])) return fail(c, DIRAC_E_NONFINITE, "non-finite V at k=%lld",
                                                                   (long long)k);
    }
    c->m = m;
    c->v_int.swap(vi);
    c->v_half.swap(vh);
    c->site_mode = false;
    c->tab_dirty = true;
    return DIRAC_OK;
}

int dirac_set_mass(dirac_ctx *c, double m) {
    if (!c) return DIRAC_E_ARG;
    if (c->v_int.empty()) return dirac_set_mass_potential_z(c, m, nullptr, nullptr, planes_of(c));
    const std::vector<double> vi = c->v_int, vh = c->v_half;
    return dirac_set_mass_potential_z(c, m, vi.data(), vh.data(), planes_of(c));
}

int dirac_set_potential_z(dirac_ctx *c, const double *v_int, const double *v_half, int64_t nz) {
    if (!c) return DIRAC_E_ARG;
    return dirac_set_mass_potential_z(c, c->m, v_int, v_half, nz);
}

int dirac_set_theta_field(dirac_ctx *c, void *const theta[]) {
    if (!c || !theta) return DIRAC_E_ARG;
    if (c->is_batch) return fail(c, DIRAC_E_STATE, "batch context");
    int narr = c->ndim == 3 ? 8 : 4;
    for (int q = 0; q < narr; ++q)
        if (!theta[q]) return fail(c, DIRAC_E_ARG, "null theta array %d", q);
    for (int q = 0; q < 8; ++q) c->theta[q] = q < narr ? theta[q] : nullptr;
    c->site_mode = true;
    return DIRAC_OK;
}

int dirac_set_links(dirac_ctx *c, void *const links[]) {
    if (!c) return DIRAC_E_ARG;
    if (c->is_batch) return fail(c, DIRAC_E_STATE, "batch context");
    if (c->zh && links) return fail(c, DIRAC_E_STATE, "links are not available in z-slab mode");
    if (c->zbc && links) return fail(c, DIRAC_E_STATE, "links are not available with DIRAC_ZERO_BC");
    for (int q = 0; q < 24; ++q) c->links[q] = nullptr;
    c->links_on = false;
    if (!links) return DIRAC_OK;
    const int nl = c->ndim == 3 ? 24 : 8;
    for (int q = 0; q < nl; ++q)
        if (!links[q]) return fail(c, DIRAC_E_ARG, "null link array %d", q);
    for (int q = 0; q < nl; ++q) c->links[q] = links[q];
    c->links_on = true;
    return DIRAC_OK;
}

int dirac_coef_from_theta_host(float *coef, const double *theta, int64_t n) {
    if (!coef || !theta || n < 0) return DIRAC_E_ARG;
    for (int64_t t = 0; t < n; ++t) {
        if (!isfinite(theta[t])) return DIRAC_E_NONFINITE;
        gamma32_search(theta[t], &coef[2 * t], &coef[2 * t + 1]);
    }
    return DIRAC_OK;
}

int dirac_coef_from_theta(void *coef, const void *theta, int64_t n, void *stream) {
    return dirac_coef_from_theta_c(coef, theta, nullptr, n, stream);
}

int dirac_coef_from_theta_c(void *coef, const void *theta, const void *theta_im, int64_t n, void *stream) {
    if (!coef || !theta || n < 0) return DIRAC_E_ARG;
    if (n == 0) return DIRAC_OK;
    if (launch_coef_from_theta(coef, (const double *)theta, (const double *)theta_im, n, (hipStream_t)stream) !=
        hipSuccess)
        return DIRAC_E_HIP;
    return DIRAC_OK;
}

int dirac_coef_from_fields(void *coef, int dtype, double dt, double sgn_m, const void *v, const void *w, int64_t n,
                           void *stream) {
    if (!coef || n < 0 || !isfinite(dt) || !isfinite(sgn_m)) return DIRAC_E_ARG;
    if (dtype != DIRAC_C64 && dtype != DIRAC_C128) return DIRAC_E_ARG;
    if (dtype == DIRAC_C128 && w) return DIRAC_E_ARG;     // complex128 records hold a real theta
    if (n == 0) return DIRAC_OK;
    if (launch_coef_from_fields(coef, dtype == DIRAC_C64, 0.5 * dt, sgn_m, (const double *)v, (const double *)w, n,
                                (hipStream_t)stream) != hipSuccess)
        return DIRAC_E_HIP;
    return DIRAC_OK;
}

int dirac_theta_from_fields(dirac_ctx *c, double m, void *const v_site[], void *const theta[], void *stream) {
    if (!c || !theta || !isfinite(m)) return DIRAC_E_ARG;
    if (c->is_batch) return fail(c, DIRAC_E_STATE, "batch context");
    int narr = c->ndim == 3 ? 8 : 4;
    for (int q = 0; q < narr; ++q)
        if (!theta[q]) return fail(c, DIRAC_E_ARG, "null theta array %d", q);
    void *th8[8] = {0}, *v8[8] = {0};
    for (int q = 0; q < narr; ++q) {
        th8[q] = theta[q];
        v8[q] = v_site ? v_site[q] : nullptr;
    }
    hipStream_t s = (hipStream_t)stream;
    int64_t ncell = c->nx * c->ny * planes_of(c);
    if (c->dtype == DIRAC_C64) HIPCHK(c, launch_theta_fields<float>(th8, v8, narr, ncell, 0.5 * c->dt, m, s));
    else HIPCHK(c, launch_theta_fields<double>(th8, v8, narr, ncell, 0.5 * c->dt, m, s));
    c->m = m;
    return dirac_set_theta_field(c, theta);
}

int dirac_set_kernel(dirac_ctx *c, int kernel, int tile_y, int zchunk) {
    if (!c) return DIRAC_E_ARG;
    if (kernel < DIRAC_KERNEL_AUTO || kernel > DIRAC_KERNEL_FUSED2) return fail(c, DIRAC_E_ARG, "bad kernel %d", kernel);
    if (tile_y != 0 && tile_y != 4 && tile_y != 8) return fail(c, DIRAC_E_ARG, "tile_y must be 0, 4 or 8");
    if (zchunk < 0) return fail(c, DIRAC_E_ARG, "zchunk must be >= 0");
    c->kernel = kernel;
    c->tile_y = tile_y;
    c->zchunk = zchunk;
    return DIRAC_OK;
}

int dirac_step(dirac_ctx *c, int64_t n, void *stream) {
    int rc = check_ready(c, !c || !c->site_mode);
    if (rc) return rc;
    if (n < 0) return fail(c, DIRAC_E_ARG, "n must be >= 0");
    rc = slab_step_check(c, n);
    if (rc) return rc;
    hipStream_t s = (hipStream_t)stream;
    return c->dtype == DIRAC_C64 ? run_steps<float>(c, n, false, s) : run_steps<double>(c, n, false, s);
}

int dirac_reverse(dirac_ctx *c, int64_t n, void *stream) {
    int rc = check_ready(c, !c || !c->site_mode);
    if (rc) return rc;
    if (c->zh) return fail(c, DIRAC_E_STATE, "z-slab contexts step forward only");
    if (n < 0) return fail(c, DIRAC_E_ARG, "n must be >= 0");
    hipStream_t s = (hipStream_t)stream;
    return c->dtype == DIRAC_C64 ? run_steps<float>(c, n, true, s) : run_steps<double>(c, n, true, s);
}

int dirac_step_norm(dirac_ctx *c, int64_t n, void *dev_out, void *stream) {
    int rc = check_ready(c, true);
    if (rc) return rc;
    if (n < 1 || !dev_out) return fail(c, DIRAC_E_ARG, "need n >= 1 and an output");
    rc = slab_step_check(c, n);
    if (rc) return rc;
    hipStream_t s = (hipStream_t)stream;
    double *part = (double *)scratch_at(c, off_partial(c));
    const size_t cap_sz = partial_doubles(c) / 2;
    const int cap = cap_sz > 0x7fffffff ? 0x7fffffff : (int)cap_sz;
    const int kc = kernel_choice(c);
    const bool fp32 = c->dtype == DIRAC_C64;
    const Route r = fp32 ? route_of<float>(c, n, Op::step_norm) : route_of<double>(c, n, Op::step_norm);
    if (r.way == Way::march3) {
        rc = upload_tables(c, s);
        if (rc) return rc;
        int nb = 0;
        rc = fp32 ? run_march3<float>(c, r.plan, false, s, part, cap, &nb)
                  : run_march3<double>(c, r.plan, false, s, part, cap, &nb);
        if (rc) return rc;
        HIPCHK(c, launch_final_sum(part, nb, 2, (double *)dev_out, s));
        return DIRAC_OK;
    }
    if (c->ndim == 3 && kc == DIRAC_KERNEL_FUSED2 && n >= 2 && !c->links_on) {
        rc = dirac_step(c, n - 2, stream);
        if (rc) return rc;
        rc = upload_tables(c, s);
        if (rc) return rc;
        int nb = 0;
        hipError_t e;
        if (c->dtype == DIRAC_C64) {
            FusedArgs<float> a = fused_args<float>(c);
            a.npart = part;
            a.npart_cap = cap;
            e = launch_two<float>(c, a, s, &nb);
        } else {
            FusedArgs<double> a = fused_args<double>(c);
            a.npart = part;
            a.npart_cap = cap;
            e = launch_two<double>(c, a, s, &nb);
        }
        if (e == hipSuccess) {
            c->cur = 1 - c->cur;
            HIPCHK(c, launch_final_sum(part, nb, 2, (double *)dev_out, s));
            return DIRAC_OK;
        }
        if (nb <= cap) HIPCHK(c, e);   // a real launch failure
        // more workgroups than partial slots (the area is sized so that this
        // does not happen).  A z-slab's halos are stale after a launch, so a
        // reduction after the step would be wrong there: refuse.  Otherwise the
        // same two steps without the in-step sum, then the reduction.
        if (c->zh) return fail(c, DIRAC_E_SHAPE, "z-slab mode: %d workgroups exceed the %d partial slots", nb, cap);
        if (c->dtype == DIRAC_C64) HIPCHK(c, launch_fused3x2<float>(fused_args<float>(c), c->site_mode, s));
        else HIPCHK(c, launch_fused3x2<double>(fused_args<double>(c), c->site_mode, s));
        c->cur = 1 - c->cur;
        double *res = (double *)scratch_at(c, off_result(c));
        rc = dirac_norm_device(c, res, stream);
        if (rc) return rc;
        HIPCHK(c, hipMemcpyAsync(dev_out, res + 1, 2 * sizeof(double), hipMemcpyDeviceToDevice, s));
        return DIRAC_OK;
    }
    const bool stepped = r.way == Way::tile2;
    if (stepped) {
        rc = upload_tables(c, s);
        if (rc) return rc;
        rc = fp32 ? run_tile2<float>(c, n, false, r.passes, s) : run_tile2<double>(c, n, false, r.passes, s);
        if (rc) return rc;
    }
    if (!stepped) {
        rc = dirac_step(c, n - 1, stream);
        if (rc) return rc;
    }
    if (c->ndim == 3 && (kc == DIRAC_KERNEL_FUSED || kc == DIRAC_KERNEL_FUSED2) && !c->links_on) {
        int nb = 0;
        hipError_t e;
        if (c->dtype == DIRAC_C64) {
            FusedArgs<float> a = fused_args<float>(c);
            a.npart = part;
            a.npart_cap = cap;
            e = launch_fused3<float>(a, c->site_mode, c->tile_y, s, &nb);
        } else {
            FusedArgs<double> a = fused_args<double>(c);
            a.npart = part;
            a.npart_cap = cap;
            e = launch_fused3<double>(a, c->site_mode, c->tile_y, s, &nb);
        }
        if (e == hipSuccess) {
            c->cur = 1 - c->cur;
            HIPCHK(c, launch_final_sum(part, nb, 2, (double *)dev_out, s));
            return DIRAC_OK;
        }
        if (nb <= cap) HIPCHK(c, e);   // a real launch failure
        if (c->zh) return fail(c, DIRAC_E_SHAPE, "z-slab mode: %d workgroups exceed the %d partial slots", nb, cap);
    }
    if (!stepped) rc = dirac_step(c, 1, stream);
    if (rc) return rc;
    double *res = (double *)scratch_at(c, off_result(c));
    rc = dirac_norm_device(c, res, stream);
    if (rc) return rc;
    HIPCHK(c, hipMemcpyAsync(dev_out, res + 1, 2 * sizeof(double), hipMemcpyDeviceToDevice, s));
    return DIRAC_OK;
}

int dirac_route(dirac_ctx *c, int64_t n, int call, char *out, size_t len) {
    if (!c || !out || len == 0) return DIRAC_E_ARG;
    out[0] = 0;
    if (c->is_batch && call != DIRAC_CALL_STEP) return fail(c, DIRAC_E_STATE, "batch context");
    if (n < 0 || call < DIRAC_CALL_STEP || call > DIRAC_CALL_STEP_NORM || (call == DIRAC_CALL_STEP_NORM && n < 1))
        return fail(c, DIRAC_E_ARG, "bad n or call");
    const std::string t = c->is_batch             ? batch_route_text(c, n)
                          : c->dtype == DIRAC_C64 ? route_text<float>(c, n, (Op)call)
                                                  : route_text<double>(c, n, (Op)call);
    if (t.size() >= len) return fail(c, DIRAC_E_SHAPE, "the text takes %zu bytes", t.size() + 1);
    memcpy(out, t.c_str(), t.size() + 1);
    return DIRAC_OK;
}

int dirac_norm_device(dirac_ctx *c, void *dev_out, void *stream) {
    int rc = check_ready(c, true);
    if (rc) return rc;
    if (!dev_out) return fail(c, DIRAC_E_ARG, "null output");
    hipStream_t s = (hipStream_t)stream;
    double *part = (double *)scratch_at(c, off_partial(c));
    if (c->links_on) {
        const LinkPtrs L = link_ptrs(c);
        if (c->dtype == DIRAC_C64) HIPCHK(c, launch_norm_links<float>(reduce_args<float>(c, 0.0), L, c->ndim, s));
        else HIPCHK(c, launch_norm_links<double>(reduce_args<double>(c, 0.0), L, c->ndim, s));
    } else if (c->dtype == DIRAC_C64) {
        ReduceArgs<float> a = reduce_args<float>(c, 0.0);
        HIPCHK(c, c->ndim == 3 ? launch_norm3<float>(a, s) : launch_norm2<float>(a, s));
    } else {
        ReduceArgs<double> a = reduce_args<double>(c, 0.0);
        HIPCHK(c, c->ndim == 3 ? launch_norm3<double>(a, s) : launch_norm2<double>(a, s));
    }
    HIPCHK(c, launch_final_sum(part, kReduceBlocks, kNormVals, (double *)dev_out, s));
    return DIRAC_OK;
}

int dirac_norm(dirac_ctx *c, double out[3], void *stream) {
    if (!out) return c ? fail(c, DIRAC_E_ARG, "null output") : DIRAC_E_ARG;
    int rc = check_ready(c, true);
    if (rc) return rc;
    double *res = (double *)scratch_at(c, off_result(c));
    rc = dirac_norm_device(c, res, stream);
    if (rc) return rc;
    hipStream_t s = (hipStream_t)stream;
    HIPCHK(c, hipMemcpyAsync(out, res, 3 * sizeof(double), hipMemcpyDeviceToHost, s));
    HIPCHK(c, hipStreamSynchronize(s));
    for (int q = 0; q < 3; ++q)
        if (!isfinite(out[q])) return fail(c, DIRAC_E_NONFINITE, "norm value %d is not finite", q);
    return DIRAC_OK;
}

int dirac_observables(dirac_ctx *c, double z0, double out[9], void *stream) {
    int rc = check_ready(c, true);
    if (rc) return rc;
    if (c->zh) return fail(c, DIRAC_E_STATE, "not available in z-slab mode (dirac_norm is)");
    if (!out || !isfinite(z0)) return fail(c, DIRAC_E_ARG, "bad output or z0");
    hipStream_t s = (hipStream_t)stream;
    double *part = (double *)scratch_at(c, off_partial(c));
    double *res = (double *)scratch_at(c, off_result(c));
    if (c->dtype == DIRAC_C64) {
        ReduceArgs<float> a = reduce_args<float>(c, z0);
        HIPCHK(c, c->ndim == 3 ? launch_obs3<float>(a, s) : launch_obs2<float>(a, s));
    } else {
        ReduceArgs<double> a = reduce_args<double>(c, z0);
        HIPCHK(c, c->ndim == 3 ? launch_obs3<double>(a, s) : launch_obs2<double>(a, s));
    }
    HIPCHK(c, launch_final_sum(part, kReduceBlocks, kObsVals, res, s));
    HIPCHK(c, hipMemcpyAsync(out, res, kObsVals * sizeof(double), hipMemcpyDeviceToHost, s));
    HIPCHK(c, hipStreamSynchronize(s));
    for (int q = 0; q < kObsVals; ++q)
        if (!isfinite(out[q])) return fail(c, DIRAC_E_NONFINITE, "observable %d is not finite", q);
    return DIRAC_OK;
}

int dirac_seed_region(dirac_ctx *c, double z0, void *const lam[], void *stream) {
    int rc = check_ready(c, false);
    if (rc) return rc;
    if (c->zh) return fail(c, DIRAC_E_STATE, "not available in z-slab mode");
    if (!lam || !isfinite(z0)) return fail(c, DIRAC_E_ARG, "bad lam or z0");
    int narr = c->ndim == 3 ? 8 : 4;
    void *l8[8] = {0};
    for (int q = 0; q < narr; ++q) {
        if (!lam[q]) return fail(c, DIRAC_E_ARG, "null lam array %d", q);
        l8[q] = lam[q];
    }
    hipStream_t s = (hipStream_t)stream;
    if (c->dtype == DIRAC_C64) {
        ReduceArgs<float> a = reduce_args<float>(c, z0);
        HIPCHK(c, c->ndim == 3 ? launch_seed3<float>(a, l8, s) : launch_seed2<float>(a, l8, s));
    } else {
        ReduceArgs<double> a = reduce_args<double>(c, z0);
        HIPCHK(c, c->ndim == 3 ? launch_seed3<double>(a, l8, s) : launch_seed2<double>(a, l8, s));
    }
    return DIRAC_OK;
}

int dirac_adjoint(dirac_ctx *c, int64_t n, void *const lam[], double z0, void *dLdV_int, void *dLdV_half,
                  void *stream) {
    int rc = dirac_seed_region(c, z0, lam, stream);
    if (rc) return rc;
    return dirac_adjoint_vz(c, n, lam, dLdV_int, dLdV_half, stream);
}

int dirac_adjoint_vz(dirac_ctx *c, int64_t n, void *const lam[], void *dLdV_int, void *dLdV_half, void *stream) {
    return dirac_adjoint_vz_work(c, n, lam, nullptr, dLdV_int, dLdV_half, stream);
}

int dirac_adjoint_uses_work(const dirac_ctx *c, int64_t n, int *uses) {
    if (!c || !uses) return DIRAC_E_ARG;
    *uses = !c->is_batch && c->bound && adjoint_on_march(c, n) ? 1 : 0;
    return DIRAC_OK;
}

int dirac_adjoint_vz_work(dirac_ctx *c, int64_t n, void *const lam[], void *const work[], void *dLdV_int,
                          void *dLdV_half, void *stream) {
    int rc = check_ready(c, true);
    if (rc) return rc;
    if (c->ndim != 3) return fail(c, DIRAC_E_STATE, "the V(z) gradient is defined for 3D lattices");
    if (c->zh) return fail(c, DIRAC_E_STATE, "not available in z-slab mode");
    if (c->site_mode) return fail(c, DIRAC_E_STATE, "needs a V(z) profile (dirac_set_mass_potential_z)");
    if (!c->w_int.empty())
        return fail(c, DIRAC_E_STATE, "the reversal-based adjoint needs a real potential (no absorbing layers)");
    if (c->links_on) return fail(c, DIRAC_E_STATE, "the V(z) gradient kernels carry no gauge links");
    if (c->zbc) return fail(c, DIRAC_E_STATE, "the V(z) gradient kernels are periodic (no DIRAC_ZERO_BC)");
    if (n < 0 || !lam || !dLdV_int || !dLdV_half) return fail(c, DIRAC_E_ARG, "bad arguments");
    for (int q = 0; q < 8; ++q)
        if (!lam[q]) return fail(c, DIRAC_E_ARG, "null lam array %d", q);
    // the march reads and writes lam, work and both buffer sets at once: no two of
    // their arrays may share memory
    const size_t bytes = array_bytes(c);
    auto meet = [bytes](const void *a, const void *b) { return ranges_meet(a, b, bytes); };
    for (int q = 0; work && q < 8; ++q) {
        if (!work[q]) return fail(c, DIRAC_E_ARG, "null work array %d", q);
        for (int p = 0; p < 8; ++p) {
            if (meet(work[q], lam[p]) || meet(work[q], c->buf[0][p]) || meet(work[q], c->buf[1][p]) ||
                (p < q && meet(work[q], work[p])))
                return fail(c, DIRAC_E_ARG, "work array %d overlaps a state, lam or work array", q);
            if (meet(lam[q], c->buf[0][p]) || meet(lam[q], c->buf[1][p]))
                return fail(c, DIRAC_E_ARG, "lam array %d overlaps a state array", q);
        }
    }
    const bool march = work && adjoint_on_march(c, n);
    hipStream_t s = (hipStream_t)stream;
    rc = upload_tables(c, s);
    if (rc) return rc;
    const int ntiles = adj_tiles3((int)c->nx, (int)c->ny);
    double *gpart = (double *)scratch_at(c, off_gpart(c));
    HIPCHK(c, launch_zero(gpart, (int64_t)ntiles * c->nz * 2, s));
    auto run = [&](auto zero) -> int {
        using R = decltype(zero);
        AdjArgs<R> a;
        memset(&a, 0, sizeof a);
        for (int q = 0; q < 8; ++q) {
            a.f[q] = c->buf[c->cur][q];
            a.lam[q] = lam[q];
        }
        size_t half = align256(tab_bytes<R>(c));
        a.tab_f = (const R *)scratch_at(c, off_tab(c));
        a.tab_r = (const R *)scratch_at(c, off_tab(c) + half);
        a.rx = (R)c->rx;
        a.ry = (R)c->ry;
        a.rz = (R)c->rz;
        a.nx = (int)c->nx;
        a.ny = (int)c->ny;
        a.nz = (int)c->nz;
        a.gpart = gpart;
        // sweeps 0, 1, 2 per backward step; sweep 2 of a step and sweep 0 of the
        // next run as one launch (sweep 3).  With a second set for lam, an even
        // number of steps go one launch each, there and back.
        const int64_t fused = march ? n & ~(int64_t)1 : 0;
        if (n > 0) HIPCHK(c, launch_adj3<R>(a, 0, s));
        for (int64_t t = 0; t < n - fused; ++t) {
            HIPCHK(c, launch_adj3<R>(a, 1, s));
            HIPCHK(c, launch_adj3<R>(a, t + 1 < n ? 3 : 2, s));
        }
        AdjMarchArgs<R> m;
        memset(&m, 0, sizeof m);
        m.rx = a.rx;
        m.ry = a.ry;
        m.rz = a.rz;
        m.nx = a.nx;
        m.ny = a.ny;
        m.nz = a.nz;
        m.gpart = gpart;
        for (int64_t t = 0; t < fused; ++t) {
            for (int q = 0; q < 8; ++q) {
                m.f[q] = c->buf[t & 1 ? 1 - c->cur : c->cur][q];
                m.fo[q] = c->buf[t & 1 ? c->cur : 1 - c->cur][q];
                m.lam[q] = t & 1 ? work[q] : lam[q];
                m.lamo[q] = t & 1 ? lam[q] : work[q];
            }
            HIPCHK(c, launch_adj_march<R>(m, a.tab_f, a.tab_r, t + 1 == fused, s));
        }
        return DIRAC_OK;
    };
    rc = c->dtype == DIRAC_C64 ? run(0.0f) : run(0.0);
    if (rc) return rc;
    HIPCHK(c, launch_adj_finish(gpart, ntiles, (int)c->nz, 0.5 * c->dt, (double *)dLdV_int, (double *)dLdV_half, s));
    return DIRAC_OK;
}

}  // extern "C"
