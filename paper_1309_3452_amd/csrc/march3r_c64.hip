// The (3+1)D register march for complex64 lattices.
#include "march3r.h"

namespace dirac {

namespace {
// Tables: 32 rows in 128 registers (one workgroup of 16 waves per CU); 16 and 8
// rows where those fill the chip better; three steps per launch with 24 or 12
// rows.  Records add 24 registers per cell: 16 rows by 8 waves, or 8.
constexpr M3Shape kTab[] = {{1, 4, 8, 1, 5.0}, {2, 2, 16, 1, 4.6}, {2, 1, 16, 1, 2.0}, {2, 1, 8, 2, 1.07},
                             {3, 3, 8, 1, 5.8}, {3, 1, 12, 1, 2.05}};
constexpr M3Shape kSite[] = {{1, 2, 8, 1, 3.6}, {2, 2, 8, 1, 3.3}, {2, 1, 8, 1, 1.25}};
constexpr int kNTab = sizeof(kTab) / sizeof(kTab[0]), kNSite = sizeof(kSite) / sizeof(kSite[0]);

const M3Pick &pick(int steps, bool site, bool zb, int nx, int ny, int nz) {
    return m3_pick(site ? kSite : kTab, site ? kNSite : kNTab, steps, site, zb, nx, ny, nz);
}
}  // namespace

template <> double march3r_us<float>(int steps, bool site, bool zb, int nx, int ny, int nz) {
    return pick(steps, site, zb, nx, ny, nz).us;
}

template <>
hipError_t launch_march3r<float>(const FusedArgs<float> &a, int steps, bool site, bool zb, hipStream_t s,
                                 int *nblocks_out) {
    const M3Pick &p = pick(steps, site, zb, a.nx, a.ny, a.nz);
    const int q = p.shape;
    if (site) {
        if (q == 0) return m3_launch<float, 1, 2, 8, 2, true>(a, p, zb, s, nblocks_out);
        if (q == 1) return m3_launch<float, 2, 2, 8, 2, true>(a, p, zb, s, nblocks_out);
        if (q == 2) return m3_launch<float, 2, 1, 8, 4, true>(a, p, zb, s, nblocks_out);
        return hipErrorInvalidValue;
    }
    if (q == 0) return m3_launch<float, 1, 4, 8, 2, false>(a, p, zb, s, nblocks_out);
    if (q == 1) return m3_launch<float, 2, 2, 16, 4, false>(a, p, zb, s, nblocks_out);
    if (q == 2) return m3_launch<float, 2, 1, 16, 4, false>(a, p, zb, s, nblocks_out);
    if (q == 3) return m3_launch<float, 2, 1, 8, 4, false>(a, p, zb, s, nblocks_out);
    if (q == 4) return m3_launch<float, 3, 3, 8, 2, false>(a, p, zb, s, nblocks_out);
    if (q == 5) return m3_launch<float, 3, 1, 12, 3, false>(a, p, zb, s, nblocks_out);
    return hipErrorInvalidValue;
}

}  // namespace dirac
