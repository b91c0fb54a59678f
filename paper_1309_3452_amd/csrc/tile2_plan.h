// Host side of the (2+1)D register tiles (tile2.hip): how a number of steps is
// split into passes, and the launch of a pass.
#pragma once

#include "internal.h"

namespace dirac {

constexpr int kTile2MaxSteps = 8;      // most steps of one pass
int resident_per_round();              // workgroups of one per CU (fused2.hip)
// What a cell carries beside its amplitudes: bit 0 per-site records, bit 1 links.
inline int tile2_kind(bool site, bool links) { return (site ? 1 : 0) | (links ? 2 : 0); }
int tile2_rows(int shape);             // rows of a tile shape's region
int64_t tile2_tiles(int shape, int ring, int64_t nx, int64_t ny);
// estimated microseconds of a pass
double tile2_pass_us(int shape, int steps, int64_t tiles, double cells, bool fp32, int kind);
// the fastest shape for a pass of `steps` over `count` lattices, and its time
int tile2_best_shape(int steps, int64_t count, const int64_t *nx, const int64_t *ny, bool fp32, int kind, double *us);
// What forming the registers of that many region cells adds to a pass.  tile2_pass_us is
// for tiles that are mostly lattice; where a region is mostly ring or periodic images (a
// few very long rows) its loads count too: 1.4 ps a region cell in complex64 without a
// potential, 1.5 in complex128, two and four times that with records, 2 and 5.6 ps with
// links.  Measured / estimated, one step: 400000 x 1 complex64 29 / 30 us, complex128 per
// site 76 / 76, with links 88 / 88, 400000 x 8 complex64 52 / 54.
inline double tile2_region_us(double region_cells, bool fp32, int kind) {
    constexpr double ps[2][4] = {{1.5, 5.5, 5.6, 9.0}, {1.4, 2.8, 2.0, 3.0}};
    return 1e-6 * ps[fp32 ? 1 : 0][kind] * region_cells;
}
// estimated microseconds of n steps in that many passes, those loads counted
double tile2_total_us(int64_t n, int64_t passes, int64_t nx, int64_t ny, bool fp32, int kind);
// passes for n steps with the parity of `parity`; 0 if there is no such split
int64_t tile2_passes(int64_t n, int parity, int64_t count, const int64_t *nx, const int64_t *ny, bool fp32, int kind);
template <typename R> hipError_t launch_tile2(const FusedArgs<R> &a, bool site, bool zb, int steps, hipStream_t s);
// The same with gauge links (tile2links.hip), periodic and forward.
template <typename R>
hipError_t launch_tile2_links(const FusedArgs<R> &a, const LinkPtrs &L, bool site, int steps, hipStream_t s);

}  // namespace dirac
