// Thin Householder QR of a matrix held in the registers of one workgroup, shared by the
// variational compression's site factorisation and the truncation's subspace refinement.
#pragma once

#include "common.h"

namespace peps {

// Column j of the m x n matrix belongs to wave j % NW (slot j / NW), its rows i = lane + 64 r
// (r < RPL) to that wave's lanes, so m <= 64 RPL and n <= NW SL; rows >= m hold zeros.  Only
// the current reflector v_k is shared, through a double-buffered LDS vector (one barrier per
// step): the owner of column k forms it with wave reductions, every wave applies it to its
// own trailing columns.  On return column k holds R above the diagonal and on it, v_k below;
// tau[k] in LDS (visible after the next barrier).
template <int NW, int SL, int RPL>
__device__ __forceinline__ void thinq_factor(double (&a)[SL][RPL], int m, int n, double (*vbuf)[64 * RPL],
                                             double* tau) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (int k = 0; k < n; ++k) {
        double* v = vbuf[k & 1];
        if (w == k % NW) {
            const int sk = k / NW;
            double x[RPL];
#pragma unroll
            for (int s = 0; s < SL; ++s)
                if (s == sk) {
#pragma unroll
                    for (int r = 0; r < RPL; ++r) x[r] = a[s][r];
                }
            double ss = 0.0, al = 0.0;
#pragma unroll
            for (int r = 0; r < RPL; ++r) {
                const int i = lane + 64 * r;
                if (i > k && i < m) ss += x[r] * x[r];
                if (i == k) al = x[r];
            }
            ss = lane_group_sum(ss, 64);
            al = lane_group_sum(al, 64);
            double tk = 0.0, beta = al, sc = 0.0;
            if (ss > 0.0) {
                beta = -copysign(sqrt(al * al + ss), al);
                tk = (beta - al) / beta;
                sc = 1.0 / (al - beta);
            }
#pragma unroll
            for (int r = 0; r < RPL; ++r) {
                const int i = lane + 64 * r;
                double vi = 0.0;
                if (i == k) {
                    vi = 1.0;
                    x[r] = beta;
                } else if (i > k && i < m) {
                    vi = ss > 0.0 ? x[r] * sc : 0.0;
                    x[r] = vi;
                }
                v[i] = vi;
            }
#pragma unroll
            for (int s = 0; s < SL; ++s)
                if (s == sk) {
#pragma unroll
                    for (int r = 0; r < RPL; ++r) a[s][r] = x[r];
                }
            if (lane == 0) tau[k] = tk;
        }
        __syncthreads();
        const double tk = tau[k];
        if (tk != 0.0) {
            double vr[RPL];
#pragma unroll
            for (int r = 0; r < RPL; ++r) vr[r] = v[lane + 64 * r];
#pragma unroll
            for (int s = 0; s < SL; ++s) {
                const int j = s * NW + w;
                if (j > k && j < n) {
                    double d = 0.0;
#pragma unroll
                    for (int r = 0; r < RPL; ++r) d += vr[r] * a[s][r];
                    d = lane_group_sum(d, 64) * tk;
#pragma unroll
                    for (int r = 0; r < RPL; ++r) a[s][r] -= d * vr[r];
                }
            }
        }
    }
}

// The explicit Q of thinq_factor in place, backwards: H_k applied to the columns right of k,
// then column k becomes e_k - tau_k v_k.  A barrier must separate the two (vbuf is reused).
template <int NW, int SL, int RPL>
__device__ __forceinline__ void thinq_form(double (&a)[SL][RPL], int m, int n, double (*vbuf)[64 * RPL],
                                           const double* tau) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (int k = n - 1; k >= 0; --k) {
        double* v = vbuf[k & 1];
        const double tk = tau[k];
        if (w == k % NW) {
            const int sk = k / NW;
#pragma unroll
            for (int s = 0; s < SL; ++s)
                if (s == sk) {
#pragma unroll
                    for (int r = 0; r < RPL; ++r) {
                        const int i = lane + 64 * r;
                        const double vi = i == k ? 1.0 : (i > k && i < m ? a[s][r] : 0.0);
                        v[i] = vi;
                        a[s][r] = i < k ? 0.0 : (i == k ? 1.0 - tk : -tk * vi);
                    }
                }
        }
        __syncthreads();
        if (tk != 0.0) {
            double vr[RPL];
#pragma unroll
            for (int r = 0; r < RPL; ++r) vr[r] = v[lane + 64 * r];
#pragma unroll
            for (int s = 0; s < SL; ++s) {
                const int j = s * NW + w;
                if (j > k && j < n) {
                    double d = 0.0;
#pragma unroll
                    for (int r = 0; r < RPL; ++r) d += vr[r] * a[s][r];
                    d = lane_group_sum(d, 64) * tk;
#pragma unroll
                    for (int r = 0; r < RPL; ++r) a[s][r] -= d * vr[r];
                }
            }
        }
    }
}

}  // namespace peps
