// The (3+1)D register march for complex64 lattices with V(z) tables.
#include "march3r.h"

namespace dirac {

namespace {
// 32 rows in 128 registers (one workgroup of 16 waves per CU); 16 and 8 rows where
// those fill the chip better; three steps per launch with 24 or 12 rows.
constexpr M3Shape kShapes[] = {{1, 4, 8, 1, 5.0}, {2, 2, 16, 1, 4.6}, {2, 1, 16, 1, 2.0}, {2, 1, 8, 2, 1.07},
                               {3, 3, 8, 1, 5.8}, {3, 1, 12, 1, 2.05}};

const M3Pick &pick(int steps, bool zb, int nx, int ny, int nz) {
    return m3_pick<float>(kShapes, sizeof(kShapes) / sizeof(kShapes[0]), steps, zb, nx, ny, nz);
}
}  // namespace

template <> double march3r_us_of<float, false>(int steps, bool zb, int nx, int ny, int nz) {
    return pick(steps, zb, nx, ny, nz).us;
}

template <>
hipError_t launch_march3r_of<float, false>(const FusedArgs<float> &a, int steps, bool zb, hipStream_t s, int *nblocks_out) {
    const M3Pick &p = pick(steps, zb, a.nx, a.ny, a.nz);
    if (p.shape == 0) return m3_launch<float, 1, 4, 8, 2, false>(a, p, zb, s, nblocks_out);
    if (p.shape == 1) return m3_launch<float, 2, 2, 16, 4, false>(a, p, zb, s, nblocks_out);
    if (p.shape == 2) return m3_launch<float, 2, 1, 16, 4, false>(a, p, zb, s, nblocks_out);
    if (p.shape == 3) return m3_launch<float, 2, 1, 8, 4, false>(a, p, zb, s, nblocks_out);
    if (p.shape == 4) return m3_launch<float, 3, 3, 8, 2, false>(a, p, zb, s, nblocks_out);
    if (p.shape == 5) return m3_launch<float, 3, 1, 12, 3, false>(a, p, zb, s, nblocks_out);
    return hipErrorInvalidValue;
}

}  // namespace dirac
