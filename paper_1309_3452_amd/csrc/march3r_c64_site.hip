// The (3+1)D register march for complex64 lattices with per-site records.
#include "march3r.h"

namespace dirac {

namespace {
// Records add 24 registers per cell: 16 rows by 8 waves, or 8.
constexpr M3Shape kShapes[] = {{1, 2, 8, 1, 3.6}, {2, 2, 8, 1, 3.3}, {2, 1, 8, 1, 1.25}};

const M3Pick &pick(int steps, bool zb, int nx, int ny, int nz) {
    return m3_pick<float>(kShapes, sizeof(kShapes) / sizeof(kShapes[0]), steps, zb, nx, ny, nz);
}
}  // namespace

template <> double march3r_us_of<float, true>(int steps, bool zb, int nx, int ny, int nz) {
    return pick(steps, zb, nx, ny, nz).us;
}

template <>
hipError_t launch_march3r_of<float, true>(const FusedArgs<float> &a, int steps, bool zb, hipStream_t s, int *nblocks_out) {
    const M3Pick &p = pick(steps, zb, a.nx, a.ny, a.nz);
    if (p.shape == 0) return m3_launch<float, 1, 2, 8, 2, true>(a, p, zb, s, nblocks_out);
    if (p.shape == 1) return m3_launch<float, 2, 2, 8, 2, true>(a, p, zb, s, nblocks_out);
    if (p.shape == 2) return m3_launch<float, 2, 1, 8, 4, true>(a, p, zb, s, nblocks_out);
    return hipErrorInvalidValue;
}

}  // namespace dirac
