// Single-lattice launches of the (2+1)D register tile (tile2.h) and the rule that
// splits a number of steps into passes, shared with the batches.
#include <math.h>

#include <algorithm>

#include "tile2.h"
#include "tile2_plan.h"

namespace dirac {

namespace {

// Blocks are dealt to the eight XCDs in turn; each XCD gets a contiguous run of
// tiles, so that neighbouring tiles find each other's ring in its L2.
__device__ __forceinline__ int tile_of_block(int b, int n) {
    const int x = b & 7, q = n >> 3, r = n & 7;
    return x * q + min(x, r) + (b >> 3);
}

template <typename R, bool SITE, bool ZB, int K, int NW>
__global__ __launch_bounds__(NW * 64, 4) void k2_tile(FusedArgs<R> a, const R *__restrict__ tab, int steps, int ring) {
    __shared__ T2Edge<R, NW> sh;
    const int L = tile_of_block(blockIdx.x, gridDim.x);
    tile2<R, SITE, ZB, K, NW>(a, tab, steps, ring, L % a.ntx, L / a.ntx, sh);
}

template <typename R, bool SITE, bool ZB>
void launch_shape(int shape, const FusedArgs<R> &a, int steps, dim3 g, hipStream_t s) {
    if (shape == 0)
        hipLaunchKernelGGL((k2_tile<R, SITE, ZB, 1, 16>), g, dim3(1024), 0, s, a, a.tab, steps, steps);
    else if (shape == 1)
        hipLaunchKernelGGL((k2_tile<R, SITE, ZB, 2, 16>), g, dim3(1024), 0, s, a, a.tab, steps, steps);
    else if constexpr (!(SITE && sizeof(R) == 8))
        hipLaunchKernelGGL((k2_tile<R, SITE, ZB, 6, 8>), g, dim3(512), 0, s, a, a.tab, steps, steps);
}

}  // namespace

int tile2_rows(int shape) { return shape == 0 ? 16 : shape == 1 ? 32 : 48; }

int64_t tile2_tiles(int shape, int ring, int64_t nx, int64_t ny) {
    const int tw = 64 - 2 * ring, th = tile2_rows(shape) - 2 * ring;
    return ((nx + tw - 1) / tw) * ((ny + th - 1) / th);
}

// Microseconds of one pass of `steps` steps over `tiles` tiles holding `cells`
// lattice cells: a launch costs 3.2; a CU evaluates a region cell in 0.66 ns
// (complex64), 0.85 ns (complex128) or 1.4 ns (complex128 per site, one workgroup
// per CU), with links 2.2 times that, counting whole rounds while there are few, 1.6 times that where eight
// waves have a CU to themselves; the bytes of one pass go at 5 TB/s, 9 out of the
// caches.  Both overlap, the longer one only in part (cube root of the sum of
// cubes: 2047 x 1531 complex64 per site measured 77, 84, 105 us for 5, 6, 7 steps
// with 62, 82, 105 us of arithmetic and 60 of bytes).
double tile2_pass_us(int shape, int steps, int64_t tiles, double cells, bool fp32, int kind) {
    const double cus = resident_per_round();
    const bool site = kind & 1, links = kind & 2;
    double per = (double)tiles / cus;
    if (per <= 4.0) per = (double)((tiles + (int64_t)cus - 1) / (int64_t)cus);
    double rows = (double)tile2_rows(shape) * steps;
    if (shape == 0) rows -= (double)steps * (steps - 1);          // the waves that skip
    const double cell_ns = (fp32 ? 0.66 : site ? 1.4 : 0.85) * (shape == 2 && per < 2.0 ? 1.6 : 1.0) * (links ? 2.2 : 1.0);
    const double comp = per * rows * 64.0 * cell_ns * 1e-3;
    const double bytes = cells * ((fp32 ? 64.0 : 128.0) + (site ? 32.0 : 0.0) + (links ? (fp32 ? 64.0 : 128.0) : 0.0));
    const double mem = bytes / (bytes > 2e8 ? 5e6 : 9e6);
    return 3.2 + cbrt(comp * comp * comp + mem * mem * mem);
}

int tile2_best_shape(int steps, int64_t count, const int64_t *nx, const int64_t *ny, bool fp32, int kind, double *us) {
    int best = -1;
    for (int shape = 0; shape < 3; ++shape) {
        if (shape == 2 && ((kind & 2) || ((kind & 1) && !fp32))) continue;      // not built: registers
        if (shape == 1 && (kind & 2) && !fp32) continue;
        if (tile2_rows(shape) - 2 * steps < 2) continue;
        int64_t tiles = 0;
        double cells = 0.0;
        for (int64_t b = 0; b < count; ++b) {
            tiles += tile2_tiles(shape, steps, nx[b], ny[b]);
            cells += (double)nx[b] * (double)ny[b];
        }
        const double t = tile2_pass_us(shape, steps, tiles, cells, fp32, kind);
        if (best < 0 || t < *us) {
            best = shape;
            *us = t;
        }
    }
    return best;
}

// n steps as passes: the count with the least total time by the figures above
// whose parity is that of `parity` (the passes ping-pong between two buffer sets,
// and the set that ends up with the state is part of the call's result); 0 where
// there is none (n = 1 with an even count).
int64_t tile2_passes(int64_t n, int parity, int64_t count, const int64_t *nx, const int64_t *ny, bool fp32, int kind) {
    int64_t best = 0;
    double best_us = 0.0, us[kTile2MaxSteps + 1] = {};
    for (int t = 1; t <= kTile2MaxSteps && t <= n; ++t) {
        if (tile2_best_shape(t, count, nx, ny, fp32, kind, &us[t]) < 0) break;
        int64_t p = (n + t - 1) / t;
        if ((p ^ parity) & 1) ++p;
        if (p > n) continue;
        const int64_t lo = n / p, more = n % p;                   // `more` passes of lo + 1 steps
        const double total = (double)(p - more) * us[lo] + (more ? (double)more * us[lo + 1] : 0.0);
        if (best == 0 || total < best_us) {
            best = p;
            best_us = total;
        }
    }
    return best;
}

double tile2_total_us(int64_t n, int64_t passes, int64_t nx, int64_t ny, bool fp32, int kind) {
    double total = 0.0;
    for (int more = 0; more < 2; ++more) {
        const int64_t count = more ? n % passes : passes - n % passes;
        if (count == 0) continue;
        const int steps = (int)(n / passes) + more;
        double us = 0.0;
        const int shape = tile2_best_shape(steps, 1, &nx, &ny, fp32, kind, &us);
        const double cells = (double)tile2_tiles(shape, steps, nx, ny) * tile2_rows(shape) * 64.0;
        total += (double)count * (us + tile2_region_us(cells, fp32, kind));
    }
    return total;
}

template <typename R>
hipError_t launch_tile2(const FusedArgs<R> &a0, bool site, bool zb, int steps, hipStream_t s) {
    FusedArgs<R> a = a0;
    if (steps < 1 || steps > kTile2MaxSteps || (!site && a.tab == nullptr)) return hipErrorInvalidValue;
    const int64_t nx = a.nx, ny = a.ny;
    double us = 0.0;
    const int shape = tile2_best_shape(steps, 1, &nx, &ny, sizeof(R) == 4, tile2_kind(site, false), &us);
    if (shape < 0) return hipErrorInvalidValue;
    const int64_t tiles = tile2_tiles(shape, steps, nx, ny);
    if (tiles > 0x7fffffff) return hipErrorInvalidValue;
    a.ntx = (a.nx + 64 - 2 * steps - 1) / (64 - 2 * steps);
    const dim3 g((unsigned)tiles);
    if (site) {
        if (zb) launch_shape<R, true, true>(shape, a, steps, g, s);
        else launch_shape<R, true, false>(shape, a, steps, g, s);
    } else {
        if (zb) launch_shape<R, false, true>(shape, a, steps, g, s);
        else launch_shape<R, false, false>(shape, a, steps, g, s);
    }
    return hipGetLastError();
}

template hipError_t launch_tile2<float>(const FusedArgs<float> &, bool, bool, int, hipStream_t);
template hipError_t launch_tile2<double>(const FusedArgs<double> &, bool, bool, int, hipStream_t);

}  // namespace dirac
