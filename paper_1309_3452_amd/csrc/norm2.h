// The (2+1)D functional of up to kNormGroup lattices in one reduction (batches).
#pragma once

#include "internal.h"

namespace dirac {

constexpr int kNormGroup = 32;         // lattices per launch: their descriptors are kernel arguments

struct Norm2Lat {
    const void *f[4];
    double r;                          // r_x = r_y, as the lattice's precision holds it
    int nx, ny;
};

// Blocks first[b] .. first[b + 1] - 1 reduce lattice b, first[count] <= kReduceBlocks.
struct Norm2Group {
    Norm2Lat lat[kNormGroup];
    int first[kNormGroup + 1];
    int count;
    double *partial;                   // [block][kNormVals]
};

// out: kNormVals doubles per lattice (device).
template <typename R> hipError_t launch_norm2_group(const Norm2Group &g, double *out, hipStream_t s);

}  // namespace dirac
