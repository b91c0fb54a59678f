// Couplings with gauge links (Sect. 4) shared by the link kernels: one coupling of a
// C,D / v row, and the (2+1)D rows.
#pragma once

#include "stencil3.h"

namespace dirac {

// One C,D coupling: the new A,B value x times the conjugate of its link factor u.
template <typename C> __device__ __forceinline__ C pr(C u, C x) { return cmul(cconj(u), x); }

enum { T2XP = 0, T2XM = 1, T2YP = 2, T2YM = 3 };

// u rows with links, one row per array (u: the array's four link factors at
// the cell, term order +x, -x, +y, -y):
//   u0: +x v0, -x v0[i-1], +y v1, -y v1[j-1];  u1: +x v1[i+1], -x v1, +y v0[j+1], -y v0
template <typename C, typename R>
__device__ __forceinline__ C u_row0(const C *u, C v0, C v0xm, C v1, C v1ym, R rx, R ry) {
    return sterm2(rx, csub(cmul(u[T2XP], v0), cmul(u[T2XM], v0xm)), -ry, csub(cmul(u[T2YP], v1), cmul(u[T2YM], v1ym)));
}
template <typename C, typename R>
__device__ __forceinline__ C u_row1(const C *u, C v1xp, C v1, C v0yp, C v0, R rx, R ry) {
    return sterm2(rx, csub(cmul(u[T2XP], v1xp), cmul(u[T2XM], v1)), -ry, csub(cmul(u[T2YP], v0yp), cmul(u[T2YM], v0)));
}
// v rows from their 8 couplings T[4 q + term] (q = v0, v1; term order +x, -x, +y, -y):
//   v0: u0(xp).-x  u0.+x  u1.-y  u1(ym).+y;   v1: u1.-x  u1(xm).+x  u0(yp).-y  u0.+y
template <typename C, typename R> __device__ __forceinline__ St2<C> v_rows(const C (&T)[8], R rx, R ry) {
    St2<C> s;
    s.s0 = sterm2(rx, csub(T[0], T[1]), ry, csub(T[2], T[3]));
    s.s1 = sterm2(rx, csub(T[4], T[5]), ry, csub(T[6], T[7]));
    return s;
}

}  // namespace dirac
