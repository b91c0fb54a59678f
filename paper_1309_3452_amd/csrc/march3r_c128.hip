// The (3+1)D register march for complex128 lattices with V(z) tables.
#include "march3r.h"

namespace dirac {

namespace {
// 16 rows by 8 waves of up to 256 registers (LDS edges take 128 KB), 8 rows, or 12
// (two steps of 200 x 168 x 152: 16 rows 0.29 ms, 8 rows 0.33, 12 rows 0.255).
constexpr M3Shape kShapes[] = {{1, 2, 8, 1, 4.8}, {2, 2, 8, 1, 3.5}, {2, 1, 8, 1, 1.4}, {2, 1, 12, 1, 2.15}};

const M3Pick &pick(int steps, bool zb, int nx, int ny, int nz) {
    return m3_pick<double>(kShapes, sizeof(kShapes) / sizeof(kShapes[0]), steps, zb, nx, ny, nz);
}
}  // namespace

template <> double march3r_us_of<double, false>(int steps, bool zb, int nx, int ny, int nz) {
    return pick(steps, zb, nx, ny, nz).us;
}

template <>
hipError_t launch_march3r_of<double, false>(const FusedArgs<double> &a, int steps, bool zb, hipStream_t s, int *nblocks_out) {
    const M3Pick &p = pick(steps, zb, a.nx, a.ny, a.nz);
    if (p.shape == 0) return m3_launch<double, 1, 2, 8, 2, false>(a, p, zb, s, nblocks_out);
    if (p.shape == 1) return m3_launch<double, 2, 2, 8, 2, false>(a, p, zb, s, nblocks_out);
    if (p.shape == 2) return m3_launch<double, 2, 1, 8, 2, false>(a, p, zb, s, nblocks_out);
    if (p.shape == 3) return m3_launch<double, 2, 1, 12, 3, false>(a, p, zb, s, nblocks_out);
    return hipErrorInvalidValue;
}

}  // namespace dirac
