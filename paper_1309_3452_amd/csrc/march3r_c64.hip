// The (3+1)D register march for complex64 lattices with V(z) tables.
#include "march3r.h"

namespace dirac {

namespace {
struct Unit {
    using R = float;
    static constexpr bool kRec = false;
    // 32 rows in 128 registers (one workgroup of 16 waves per CU), 5 of them spilled, with
    // the functional 14, with it and zero values outside 143 (that launch's estimate does
    // not know); 16 and 8 rows where those fill the chip better; three steps per launch with
    // 24 rows (256 registers, 14 to 16 spilled) or 12.
    static constexpr M3Shape kShapes[] = {{1, 4, 8, 2, 1, 5.0}, {2, 2, 16, 4, 1, 4.6}, {2, 1, 16, 4, 1, 2.0},
                                          {2, 1, 8, 4, 2, 1.07}, {3, 3, 8, 2, 1, 5.8}, {3, 1, 12, 3, 1, 2.05}};
};
}  // namespace

M3_UNIT(Unit)

}  // namespace dirac
