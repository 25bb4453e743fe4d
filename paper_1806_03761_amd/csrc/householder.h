// Householder scalars shared by the float64 factorisation kernels.
#pragma once

#include "common.h"

namespace peps {

// 1/sqrt(s2) and the norm sqrt(s2), from the hardware estimate with two Newton steps and one
// correction (s2 well inside the range of doubles)
__device__ __forceinline__ void hh_norm(double s2, double& rinv, double& nrm) {
    double r = __builtin_amdgcn_rsq(s2);
    r = fma(fma(-s2 * r, r, 1.0), 0.5 * r, r);
    r = fma(fma(-s2 * r, r, 1.0), 0.5 * r, r);
    const double y = s2 * r;
    nrm = fma(fma(-y, y, s2), 0.5 * r, y);
    rinv = r;
}
__device__ __forceinline__ double hh_rcp(double d) {
    double q = __builtin_amdgcn_rcp(d);
    q = fma(fma(-d, q, 1.0), q, q);
    return fma(fma(-d, q, 1.0), q, q);
}

// Column with pivot entry al and squared norm sq below it (dlarfg: beta = -sign(al) norm,
// tau = (beta - al) / beta, v = x / (al - beta)) from one reciprocal square root and one
// reciprocal: half the dependent chain of a square root and two divisions.
__device__ __forceinline__ void hh_scalars(double al, double sq, double& tk, double& be, double& sc) {
    const double s2 = fma(al, al, sq);
    if (sq == 0.0) {
        tk = 0.0;
        be = al;
        sc = 0.0;
    } else if (s2 > 1e-280 && s2 < 1e280) {
        double r, nrm;
        hh_norm(s2, r, nrm);
        const double den = fabs(al) + nrm;
        be = -copysign(nrm, al);
        sc = copysign(hh_rcp(den), al);
        tk = den * r;
    } else {
        be = -copysign(sqrt(s2), al);
        tk = (be - al) / be;
        sc = 1.0 / (al - be);
    }
}

// The same reflector unnormalised, H = I - t u u^T with u = (al - beta, x): beta, u's pivot entry
// and t = 1 / (norm (norm + |al|)).  False, through one scalar branch (al and sq are the same in every
// lane), where the squared norm is near the ends of the range of doubles.
__device__ __forceinline__ bool hh_unnormalised(double al, double sq, double& be, double& up, double& t) {
    const double s2 = fma(al, al, sq);
    double r, nrm;
    hh_norm(s2, r, nrm);
    const double den = fabs(al) + nrm;
    const bool none = sq == 0.0;
    be = none ? al : -copysign(nrm, al);
    up = none ? 0.0 : copysign(den, al);
    t = none ? 0.0 : r * hh_rcp(den);
    return !__builtin_amdgcn_readfirstlane(!none && !(s2 > 1e-280 && s2 < 1e280));
}

}  // namespace peps
