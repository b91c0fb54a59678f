// Entries of the V(z) coefficient tables: the Cayley factors of the time-averaged
// mass and potential term (Eqs. ss1-ss4), from one source for host and device.
#pragma once

#include "cayley32.h"

namespace dirac {

// FP64 Cayley coefficients, every operation rounded on its own.
__host__ __device__ inline void cayley64(double th, double out[4]) {
#pragma clang fp contract(off)
    double t2 = th * th;
    double d = 1.0 + t2;
    out[0] = (1.0 - t2) / d;
    out[1] = -((2.0 * th) / d);
    out[2] = 1.0 / d;
    out[3] = -(th / d);
}

// FP32 increment-form coefficients: gamma = 2 i th / (1 + i th) by the
// unit-modulus rounding shared with the device records (cayley32.h), beta =
// 1 / (1 + i th) rounded from FP64.
__host__ __device__ inline void cayley32(double th, float out[4]) {
#pragma clang fp contract(off)
    const double d = 1.0 + th * th;
    gamma32_search(th, &out[0], &out[1]);
    out[2] = (float)(1.0 / d);
    out[3] = (float)(-th / d);
}

// Complex theta = th + i thi (a complex potential; Im V damps for Im V < 0):
// with 1 + i theta = (1 - thi) + i th and 1 - i theta = (1 + thi) - i th,
//   beta = ((1 - thi) - i th)/den,  alpha = ((1 - thi^2 - th^2) - 2 i th)/den,
//   den = (1 - thi)^2 + th^2.
__host__ __device__ inline void cayley64c(double th, double thi, double out[4]) {
#pragma clang fp contract(off)
    if (thi == 0.0) {
        cayley64(th, out);
        return;
    }
    const double den = (1.0 - thi) * (1.0 - thi) + th * th;
    out[0] = (1.0 - thi * thi - th * th) / den;
    out[1] = -((2.0 * th) / den);
    out[2] = (1.0 - thi) / den;
    out[3] = -(th / den);
}
// FP32 increment form for a complex theta: gamma = 1 - alpha and beta rounded
// from FP64 (|alpha| != 1, so the unit-modulus search does not apply).
__host__ __device__ inline void cayley32c(double th, double thi, float out[4]) {
#pragma clang fp contract(off)
    if (thi == 0.0) {
        cayley32(th, out);
        return;
    }
    double c[4];
    cayley64c(th, thi, c);
    out[0] = (float)(1.0 - c[0]);
    out[1] = (float)(-c[1]);
    out[2] = (float)c[2];
    out[3] = (float)c[3];
}

// n complex64 entries in place: each holds its theta (two doubles, Re and Im).
hipError_t launch_table32(void *tab, int64_t n, hipStream_t s);

}  // namespace dirac
