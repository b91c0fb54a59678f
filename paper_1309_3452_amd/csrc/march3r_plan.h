// Host side of the (3+1)D register march (march3r.h): the launch of 1, 2 or 3
// steps and its estimated time.
#pragma once

#include "internal.h"

namespace dirac {

int resident_per_round();              // workgroups of one per CU (fused2.hip)
// Most steps of one launch: three only with V(z) tables in complex64.
inline int march3r_most(bool fp32, bool site) { return fp32 && !site ? 3 : 2; }
// How a launch of some steps runs: which built shape (-1: none has that many
// steps) of K rows in each of NW waves, tile width, tiles in y, chunks in z, whether
// rows wrap within the wave, and its estimated microseconds.
struct M3Pick {
    int shape = -1, K = 0, NW = 0, tw = 0, nty = 0, nzc = 0;
    bool xp = false;
    double us = 0.0;
};
// REC: with per-site records.
template <typename R, bool REC> const M3Pick &march3r_pick_of(int steps, bool zb, int nx, int ny, int nz);
template <typename R> const M3Pick &march3r_pick(int steps, bool site, bool zb, int nx, int ny, int nz) {
    return site ? march3r_pick_of<R, true>(steps, zb, nx, ny, nz) : march3r_pick_of<R, false>(steps, zb, nx, ny, nz);
}
template <typename R> double march3r_us(int steps, bool site, bool zb, int nx, int ny, int nz) {
    return march3r_pick<R>(steps, site, zb, nx, ny, nz).us;
}
// The same for two steps of the LDS march on complex64 lattices of even width
// (fused2.hip): its workgroups spend about 3.3 us on a plane, 5.4 with records.
inline double march_lds_us(bool site, int nx, int ny, int nz) {
    const int64_t tiles = (int64_t)((nx + 63) / 64) * ((ny + 7) / 8), cus = resident_per_round();
    const int nzc = pick_chunks(tiles, nz, 6);
    return 2.0 + (double)((tiles * nzc + cus - 1) / cus) * ((nz + nzc - 1) / nzc + 6) *
                     (site ? 5.4 : 3.3);
}
// One step of the LDS march's one-step kernel (fused.hip), rows of even width or
// complex128: its workgroups spend 4.3 us (complex128 3.8) on a plane of empty tiles and
// 2.6 (2.8) more on one of full ones, with records 4.9 (4.6) and 4.6 (5.0) more, and fill
// their pipeline in 10.  Measured / estimated: complex64 16 x 200 x 200 107 / 104 us, 70^3
// 28 / 29, 128^3 68 / 67, 200 x 168 x 152 181 / 176, with records 241 / 233, complex128
// 33 x 40 x 50 15 / 17, 200 x 168 x 152 319 / 317, with records 441 / 446.
inline double fused3_us(bool fp32, bool site, int nx, int ny, int nz) {
    const int w = fp32 ? 128 : 64;
    const int64_t tiles = (int64_t)((nx + w - 1) / w) * ((ny + 7) / 8), cus = resident_per_round();
    const int nzc = pick_chunks(tiles, nz, 3);
    const double full = (double)nx * ny / ((double)tiles * w * 8);
    const double plane = site ? (fp32 ? 4.9 + 4.6 * full : 4.6 + 5.0 * full) : (fp32 ? 4.3 + 2.6 * full : 3.8 + 2.8 * full);
    return 2.0 + (double)((tiles * nzc + cus - 1) / cus) * (((nz + nzc - 1) / nzc) * plane + 10.0);
}
// And on complex128 lattices with V(z) tables of at most 16 columns, half a tile of the
// LDS march: its planes take 2.0 us there, 2.4 with 16 columns (3.5 to 4.4 with more),
// where a register march iteration costs much the same whatever the row holds.  Two
// steps, LDS / register march: 1 x 200 x 200 50 / 72 us, 8 x 200 x 200 55 / 72, 16 x 200 x 200
// 62 / 72, 20 x 200 x 200 102 / 80; 1 x 64 x 256 29 / 36, 1 x 7 x 600 24 / 18.  The register
// march's estimate is a third above its time on such rows.
inline bool march_lds_wins_narrow(double march_us, int nx, int ny, int nz) {
    if (nx > 16) return false;
    const int64_t tiles = (ny + 7) / 8, cus = resident_per_round();
    const int nzc = pick_chunks(tiles, nz, 6);
    const double plane = 2.0 + 0.05 * (nx > 8 ? nx - 8 : 0);
    return 2.0 + (double)((tiles * nzc + cus - 1) / cus) * ((nz + nzc - 1) / nzc + 6) * plane < 0.75 * march_us;
}
// One launch of `steps` steps, in -> out, forward or (a.rev) of the reversed
// sequence.  With a.npart (one or two steps, forward) the per-workgroup sums of
// the functional go there.
template <typename R, bool REC>
hipError_t launch_march3r_of(const FusedArgs<R> &a, int steps, bool zb, hipStream_t s, int *nblocks_out);
template <typename R>
hipError_t launch_march3r(const FusedArgs<R> &a, int steps, bool site, bool zb, hipStream_t s, int *nblocks_out = nullptr) {
    return site ? launch_march3r_of<R, true>(a, steps, zb, s, nblocks_out)
                : launch_march3r_of<R, false>(a, steps, zb, s, nblocks_out);
}

}  // namespace dirac
