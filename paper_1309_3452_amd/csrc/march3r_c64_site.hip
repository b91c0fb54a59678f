// The (3+1)D register march for complex64 lattices with per-site records.
#include "march3r.h"

namespace dirac {

namespace {
struct Unit {
    using R = float;
    static constexpr bool kRec = true;
    // Records add 24 registers per cell: 16 rows by 8 waves, or 8 (which spill 31 with the
    // functional and zero values outside).
    static constexpr M3Shape kShapes[] = {{1, 2, 8, 2, 1, 3.6}, {2, 2, 8, 2, 1, 3.3}, {2, 1, 8, 4, 1, 1.25}};
};
}  // namespace

M3_UNIT(Unit)

}  // namespace dirac
