// The (3+1)D register march for complex128 lattices.
#include "march3r.h"

namespace dirac {

namespace {
// Tables: 16 rows by 8 waves of up to 256 registers (LDS edges take 128 KB), 8 rows,
// or 12 (64^3, two steps: 28.3 against 30.5 us with 8 rows).  Records: 8 rows, whose
// 248 registers keep each coefficient from its first use to its second; 12 waves
// that form it twice measured 227 against 218 us per step at 200 x 168 x 152.
constexpr M3Shape kTab[] = {{1, 2, 8, 1, 4.8}, {2, 2, 8, 1, 3.5}, {2, 1, 8, 1, 1.4}, {2, 1, 12, 1, 2.15}};
constexpr M3Shape kSite[] = {{1, 2, 8, 1, 5.6}, {2, 1, 8, 1, 2.15}};
constexpr int kNTab = sizeof(kTab) / sizeof(kTab[0]), kNSite = sizeof(kSite) / sizeof(kSite[0]);

const M3Pick &pick(int steps, bool site, bool zb, int nx, int ny, int nz) {
    return m3_pick(site ? kSite : kTab, site ? kNSite : kNTab, steps, site, zb, nx, ny, nz);
}
}  // namespace

template <> double march3r_us<double>(int steps, bool site, bool zb, int nx, int ny, int nz) {
    return pick(steps, site, zb, nx, ny, nz).us;
}

template <>
hipError_t launch_march3r<double>(const FusedArgs<double> &a, int steps, bool site, bool zb, hipStream_t s,
                                  int *nblocks_out) {
    const M3Pick &p = pick(steps, site, zb, a.nx, a.ny, a.nz);
    const int q = p.shape;
    if (site) {
        if (q == 0) return m3_launch<double, 1, 2, 8, 2, true>(a, p, zb, s, nblocks_out);
        if (q == 1) return m3_launch<double, 2, 1, 8, 2, true>(a, p, zb, s, nblocks_out);
        return hipErrorInvalidValue;
    }
    if (q == 0) return m3_launch<double, 1, 2, 8, 2, false>(a, p, zb, s, nblocks_out);
    if (q == 1) return m3_launch<double, 2, 2, 8, 2, false>(a, p, zb, s, nblocks_out);
    if (q == 2) return m3_launch<double, 2, 1, 8, 2, false>(a, p, zb, s, nblocks_out);
    if (q == 3) return m3_launch<double, 2, 1, 12, 3, false>(a, p, zb, s, nblocks_out);
    return hipErrorInvalidValue;
}

}  // namespace dirac
