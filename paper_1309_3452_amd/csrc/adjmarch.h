// The adjoint's backward step as one launch (adjmarch.hip), and what it shares with
// the in-place sweeps (adjoint.hip).
#pragma once

#include "device.h"
#include "internal.h"

namespace dirac {

__device__ __forceinline__ double2 alpha_of(const Coef<double> &k) { return k.c1; }
__device__ __forceinline__ float2 alpha_of(const Coef<float> &k) { return mk2(1.0f - k.c1.x, -k.c1.y); }

// conj(b) * z
template <typename C> __device__ __forceinline__ C cmulc(C b, C z) { return cmul(cconj(b), z); }

// One backward step, in -> out: state and adjoint, both ping-pong.
template <typename R> struct AdjMarchArgs {
    const void *f[8], *lam[8];
    void *fo[8], *lamo[8];
    R rx, ry, rz;
    int nx, ny, nz;
    int ntx, nty, zchunk;
    double *gpart;        // [tile][nz][2], added to
};

// Tiles of the march in x and y: its slots per plane of gpart.
int adj_march_tiles(int nx, int ny);
// Whether it is the faster way for this lattice.
bool adj_march_wins(bool fp32, int nx, int ny, int nz);
// Sweeps 1 and 3 of one backward step (last: 1 and 2).  A plane is below 4 GiB.
template <typename R>
hipError_t launch_adj_march(const AdjMarchArgs<R> &a, const R *tab_f, const R *tab_r, bool last, hipStream_t s);

}  // namespace dirac
