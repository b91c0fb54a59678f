// The (3+1)D register march for complex128 lattices with V(z) tables.
#include "march3r.h"

namespace dirac {

namespace {
struct Unit {
    using R = double;
    static constexpr bool kRec = false;
    // 16 rows by 8 waves of up to 256 registers (LDS edges take 128 KB), 8 rows, or 12
    // (two steps of 200 x 168 x 152: 16 rows 0.29 ms, 8 rows 0.33, 12 rows 0.255).  One
    // step: zero values outside only.
    static constexpr M3Shape kShapes[] = {{1, 2, 8, 2, 1, 4.8}, {2, 2, 8, 2, 1, 3.5}, {2, 1, 8, 2, 1, 1.4},
                                          {2, 1, 12, 3, 1, 2.15}};
};
}  // namespace

M3_UNIT(Unit)

}  // namespace dirac
