// Thin Householder QR of a matrix held in the registers of one workgroup, shared by the
// variational compression's site factorisation and the truncation's subspace refinement.
//
// Bound by its chain of 2 n dependent steps (LDS read, dot products, lane sums, scalars, LDS
// write, barrier).  So the slots of a wave are walked by an unrolled loop (register indexes
// known at compile time, finished slots left out), every slot's update is one run of
// straight-line code with its lane sums taken together, the scalars come from one reciprocal
// square root and one reciprocal, and on the way back the next reflector is already on its way.
// With a branch, six lane sums and two divisions per slot and step: 216 x 36 62 us, 512 x 32
// 75 us (16 waves); so 39 us and 43 us (8 waves).
#pragma once

#include "common.h"
#include "householder.h"

namespace peps {

// a's sum over the two wave halves in the lower 32 lanes, b's in the upper; and, on rows of 16
// lanes, a's sum over a pair of rows in the even one, b's in the odd one
__device__ __forceinline__ double swap32_sum(double a, double b) {
    const long long va = __double_as_longlong(a), vb = __double_as_longlong(b);
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)va, (unsigned)vb, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(va >> 32), (unsigned)(vb >> 32), false, false);
    return __longlong_as_double(((long long)hi[0] << 32) | lo[0]) +
           __longlong_as_double(((long long)hi[1] << 32) | lo[1]);
}
__device__ __forceinline__ double swap16_sum(double a, double b) {
    const long long va = __double_as_longlong(a), vb = __double_as_longlong(b);
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)va, (unsigned)vb, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(va >> 32), (unsigned)(vb >> 32), false, false);
    return __longlong_as_double(((long long)hi[0] << 32) | lo[0]) +
           __longlong_as_double(((long long)hi[1] << 32) | lo[1]);
}
// the values of lane rows 0 .. 3, each in all four
__device__ __forceinline__ void spread_rows(double v, double (&f)[4]) {
    const long long b = __double_as_longlong(v);
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)b, (unsigned)b, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const auto l2 = __builtin_amdgcn_permlane16_swap(lo[h], lo[h], false, false);
        const auto h2 = __builtin_amdgcn_permlane16_swap(hi[h], hi[h], false, false);
#pragma unroll
        for (int r = 0; r < 2; ++r) f[2 * h + r] = __longlong_as_double(((long long)h2[r] << 32) | l2[r]);
    }
}

// Wave sums of N values per lane, in place and in every lane: four at a time, each on a row of 16
// lanes of its own, in half the instructions of four separate sums; a rest of one by itself.
template <int N>
__device__ __forceinline__ void wave_sums(double (&d)[N]) {
#pragma unroll
    for (int i = 0; i < N; i += 4) {
        if (N - i == 1) {
            d[i] = lane_group_sum(d[i], 64);
        } else {
            double g = swap16_sum(swap32_sum(d[i], i + 2 < N ? d[i + 2 < N ? i + 2 : i] : 0.0),
                                  swap32_sum(d[i + 1 < N ? i + 1 : i], i + 3 < N ? d[i + 3 < N ? i + 3 : i] : 0.0));
            double f[4];
            spread_rows(lane_group_sum(g, 16), f);
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (i + u < N) d[i + u < N ? i + u : i] = f[u];
        }
    }
}

// a[s] -= tk (v . a[s]) v for the slots S0 .. of columns right of k
template <int NW, int SL, int RPL, int S0>
__device__ __forceinline__ void thinq_apply(double (&a)[SL][RPL], const double* v, double tk, int k, int lane, int w) {
    double vr[RPL], d[SL - S0];
#pragma unroll
    for (int r = 0; r < RPL; ++r) vr[r] = v[lane + 64 * r];
#pragma unroll
    for (int s = S0; s < SL; ++s) {
        double x = vr[0] * a[s][0];
#pragma unroll
        for (int r = 1; r < RPL; ++r) x = fma(vr[r], a[s][r], x);
        d[s - S0] = x;
    }
    wave_sums<SL - S0>(d);
#pragma unroll
    for (int s = S0; s < SL; ++s) {
        const double f = s * NW + w > k ? -tk * d[s - S0] : 0.0;
#pragma unroll
        for (int r = 0; r < RPL; ++r) a[s][r] = fma(f, vr[r], a[s][r]);
    }
}

template <int NW, int SL, int RPL, int S>
__device__ __forceinline__ void thinq_factor_from(double (&a)[SL][RPL], int n, double (*vbuf)[64 * RPL], double* tau,
                                                  int lane, int w) {
    if constexpr (S < SL) {
        const int c = min(NW, n - S * NW);
        for (int o = 0; o < c; ++o) {
            const int k = S * NW + o;   // column k: slot S of wave o
            double* v = vbuf[k & 1];
            if (w == o) {
                double ss = lane > k ? a[S][0] * a[S][0] : 0.0;   // n <= 64: the pivot is in the first rows
#pragma unroll
                for (int r = 1; r < RPL; ++r) ss = fma(a[S][r], a[S][r], ss);
                const long long x0 = __double_as_longlong(a[S][0]);
                const double al = __longlong_as_double(
                    ((long long)__builtin_amdgcn_readlane((int)(x0 >> 32), k) << 32) |
                    (unsigned)__builtin_amdgcn_readlane((int)x0, k));
                double tk, be, sc;
                hh_scalars(al, lane_group_sum(ss, 64), tk, be, sc);
#pragma unroll
                for (int r = 0; r < RPL; ++r) {
                    const double vi = a[S][r] * sc;
                    if (r == 0) {
                        v[lane] = lane > k ? vi : (lane == k ? 1.0 : 0.0);
                        a[S][0] = lane > k ? vi : (lane == k ? be : a[S][0]);
                    } else {
                        v[lane + 64 * r] = a[S][r] = vi;
                    }
                }
                if (lane == 0) tau[k] = tk;
            }
            __syncthreads();
            thinq_apply<NW, SL, RPL, S>(a, v, tau[k], k, lane, w);
        }
        thinq_factor_from<NW, SL, RPL, S + 1>(a, n, vbuf, tau, lane, w);
    }
}

// Column j of the m x n matrix belongs to wave j % NW (slot j / NW), its rows i = lane + 64 r
// (r < RPL) to that wave's lanes, so m <= 64 RPL and n <= NW SL <= 64; rows >= m hold zeros.
// Only the current reflector v_k is shared, through a double-buffered LDS vector (one barrier
// per step): the owner of column k forms it with wave reductions, every wave applies it to its
// own trailing columns.  On return column k holds R above the diagonal and on it, v_k below;
// tau[k] in LDS (visible after the next barrier).
template <int NW, int SL, int RPL>
__device__ __forceinline__ void thinq_factor(double (&a)[SL][RPL], int n, double (*vbuf)[64 * RPL], double* tau) {
    static_assert(NW * SL <= 64, "pivot rows");
    thinq_factor_from<NW, SL, RPL, 0>(a, n, vbuf, tau, threadIdx.x & 63, threadIdx.x >> 6);
}

// v_k, stored below the diagonal of its column, to LDS
template <int RPL>
__device__ __forceinline__ void thinq_send(const double (&x)[RPL], double* v, int k, int lane) {
    v[lane] = lane > k ? x[0] : (lane == k ? 1.0 : 0.0);
#pragma unroll
    for (int r = 1; r < RPL; ++r) v[lane + 64 * r] = x[r];
}
template <int NW, int SL, int RPL, int S>
__device__ __forceinline__ void thinq_form_from(double (&a)[SL][RPL], int n, double (*vbuf)[64 * RPL],
                                                const double* tau, int lane, int w) {
    if constexpr (S >= 0) {
        for (int o = min(NW, n - S * NW) - 1; o >= 0; --o) {
            const int k = S * NW + o;
            const double tk = tau[k];
            __syncthreads();
            // the next reflector, on its way during this one's update (its buffer was last read
            // before the barrier)
            double* vn = vbuf[(k & 1) ^ 1];
            double x[RPL];
#pragma unroll
            for (int r = 0; r < RPL; ++r) x[r] = o > 0 ? a[S][r] : a[S > 0 ? S - 1 : 0][r];
            if (k > 0 && w == (o > 0 ? o : NW) - 1) thinq_send<RPL>(x, vn, k - 1, lane);
            thinq_apply<NW, SL, RPL, S>(a, vbuf[k & 1], tk, k, lane, w);
            if (w == o) {
                a[S][0] = lane > k ? -tk * a[S][0] : (lane == k ? 1.0 - tk : 0.0);
#pragma unroll
                for (int r = 1; r < RPL; ++r) a[S][r] *= -tk;
            }
        }
        thinq_form_from<NW, SL, RPL, S - 1>(a, n, vbuf, tau, lane, w);
    }
}

// The explicit Q of thinq_factor in place, backwards: H_k applied to the columns right of k,
// then column k becomes e_k - tau_k v_k.  A barrier must separate the two (vbuf is reused).
template <int NW, int SL, int RPL>
__device__ __forceinline__ void thinq_form(double (&a)[SL][RPL], int n, double (*vbuf)[64 * RPL], const double* tau) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int k = n - 1;
    double x[RPL];
#pragma unroll
    for (int r = 0; r < RPL; ++r) {
        x[r] = a[0][r];
#pragma unroll
        for (int s = 1; s < SL; ++s) {
            asm volatile("" : "+v"(x[r]));   // selects, not an indexed copy in scratch memory
            x[r] = k / NW == s ? a[s][r] : x[r];
        }
    }
    if (w == k % NW) thinq_send<RPL>(x, vbuf[k & 1], k, lane);
    thinq_form_from<NW, SL, RPL, SL - 1>(a, n, vbuf, tau, lane, w);
}

}  // namespace peps
