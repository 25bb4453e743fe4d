// Truncation of one centre in float64: from the centre matrix M (mp x np, row-major) to the new
// boundary tensor V^T, the leading tk = min(Dc, mp, np) right singular vectors of M, and the
// carried right part H = F V.
//
// The right-to-left sweep needs neither the Q factors of the left-to-right one nor singular
// values: with R the triangular factor left of site j (from the QR sweep), F the site's raw
// tensor contracted with the kept right part H of site j+1, the centre is M = R F and the next
// right part is H' = F V.  Only the subspace spanned by the rows of V^T enters the result, and the
// centre needs four products instead of the application of Q.
// Rounding, against the sweep that carries U Sigma and applies Q: on lattices up to 16x16 at D <= 4
// and 10x6 at D = 6, random, decaying and gauge-dressed, ln|W| moved by 1e-16 .. 3e-12, that sweep's
// own noise.  On 16x16, D = 6, random, W is small by cancellation in a few configurations, where any
// float64 sweep moves far: the two differ by more than x in a share of 1.1e-10 / x of 163,840
// configurations (by up to 2e-5).  Under compensated scalings of the sites this one moves by 4e-11
// (median), the other by 8e-11; at twelve of their largest differences, 7e-7 to 2e-5, this one was
// the nearer to an extended-precision value ten times.
//
//   launch_mgemm      Gram matrix A = M^T M or M M^T, the smaller (order ns)
//   k_tr_tridiag      Householder tridiagonalisation in registers (orders up to 224)
//   k_tr_tridiag_mem  the same, blocked, with the matrix in memory (orders up to 512)
//   k_eig_tri         eigenvalues and tridiagonal eigenvectors
//   k_tr_vec          orthonormalisation, back-transformation, refinement, V^T and H
#include "common.h"
#include "householder.h"
#include "kernels.h"
#include "thinq.h"

namespace peps {

namespace {

typedef double d4v __attribute__((ext_vector_type(4)));

struct TruncLayout {
    int ns, tk, gram_right, lda, ldx;
    long long oM, oA, oD, oE, oT, oX, oL, oY, total;
};

__host__ __device__ inline TruncLayout trunc_layout(int mp, int np, int Dc) {
    TruncLayout L;
    L.gram_right = np <= mp;                 // A = M^T M, else M M^T
    L.ns = L.gram_right ? np : mp;
    L.tk = Dc < L.ns ? Dc : L.ns;
    L.lda = L.ns;
    L.ldx = L.ns;
    L.oM = 0;
    L.oA = L.oM + (long long)mp * np;
    L.oD = L.oA + (long long)L.lda * L.ns;
    L.oE = L.oD + L.ns;
    L.oT = L.oE + L.ns;
    L.oX = L.oT + L.ns;
    L.oL = L.oX + (long long)L.ldx * L.tk;
    L.oY = L.oL + L.tk;                      // mp x tk block of the refinement
    L.total = L.oY + (long long)mp * L.tk;
    return L;
}

// A Gram matrix (n x n, n at most NT threads) scaled to a trace of order one where the squares of its
// entries would leave the range of doubles.  A power of two moves no mantissa, and only ratios of the
// eigenvalues are used, so M may hold entries up to 1e154, or none above 1e-154.  Done in memory
// before the matrix is loaded: on the registers it cost them (order 216: 1.94 -> 2.08 ms a launch of
// 1024 matrices).  red: LDS, a double per wave.
template <int NT>
__device__ __forceinline__ void gram_scale(double* A, int n, double* red) {
    double trace = lane_group_sum(ld_or0((int)threadIdx.x < n, A, (int)threadIdx.x * (n + 1)), 64);
    if constexpr (NT > 64) {
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = trace;
        __syncthreads();
        trace = red[0];
#pragma unroll
        for (int i = 1; i < NT / 64; ++i) trace += red[i];
    }
    const bool far = trace > 0x1p400 || (trace > 0.0 && trace < 0x1p-400);
    if (!__builtin_amdgcn_readfirstlane(far && trace < INFINITY)) return;
    const int ex = -__builtin_amdgcn_frexp_exp(trace);
    __syncthreads();
    for (int i = threadIdx.x; i < n * n; i += NT) A[i] = __builtin_amdgcn_ldexp(A[i], ex);
    __syncthreads();
}

// ---------------------------------------------------------------------------
// tridiagonalisation in registers
// ---------------------------------------------------------------------------
// A <- H_k A H_k step by step, A (order ns <= GR NR = GC NC, full storage) in the registers of a
// GR x GC thread grid: thread (ti, tj) holds the rows ti + GR u and columns tj + GC w.  The
// cyclic layout keeps the work balanced as the trailing matrix shrinks, and the steps whose
// finished columns fill W0 column blocks run as one phase with the blocks below U0 and W0
// left out at compile time, 0.4 of the work of the full square.  Step k:
//   p = tau A v, row sums reduced over the GC lanes of a row group; w = p - (tau/2)(p.v) v;
//   A -= v w^T + w v^T; then the row group of row k+1 forms the next reflector from it.
// Two barriers per step; v and tau are double-buffered, so the next pivot can run while other
// waves finish their update.  Reflector k (unit entry at k+1) goes to row k of Am beyond k+1,
// d, e and tau to their slots.  The step is bound by its dependent chain (LDS exchange, lane
// sums, pivot scalars).  With square register blocks that never shrink and plain divisions:
// order 64, 4096 matrices 370 us, one matrix 110 us; order 216, 256 matrices 1060 us.  So: 187,
// 65 and 488 us.
template <int NR, int NC, int GR, int GC>
struct Tridiag {
    static constexpr int W = GR * NR, NW = (GR * GC + 63) / 64;
    static constexpr bool KEEP = NR * NC <= 64;   // column entries of v held in registers too
    static_assert(GR * NR == GC * NC && GR % GC == 0 && GC <= 16, "coverage");
    double A[NR][NC];
    double *Am, *e, *tau, *vb, *pb, *s_tau, *s_red;
    int ns, lda, ti, tj;

    // reflector kp from row kp (the row group ti == kp % GR, whose row block is U0)
    template <int U0, int W0>
    __device__ __forceinline__ void pivot(int kp) {
        constexpr int WZ = U0 * GR / GC;
        double s0 = 0.0, al = 0.0;
#pragma unroll
        for (int w = W0; w < NC; ++w) {
            const int j = tj + GC * w;
            const double x = A[U0][w];
            s0 = fma(j >= kp + 2 ? x : 0.0, x, s0);
            al = j == kp + 1 ? x : al;
        }
        s0 = lane_group_sum(s0, GC);
        al = lane_group_sum(al, GC);
        double tk, be, sc;
        hh_scalars(al, s0, tk, be, sc);
        double* v = vb + (kp & 1) * W;
#pragma unroll
        for (int w = WZ; w < NC; ++w) {
            const int j = tj + GC * w;
            const double x = j >= kp + 2 ? sc * A[U0][w] : (j == kp + 1 ? 1.0 : 0.0);
            v[j] = x;
            if (w >= W0 && j >= kp + 2 && j < ns) Am[(long long)kp * lda + j] = x;
        }
        if (tj == 0) {
            s_tau[kp & 1] = tk;
            tau[kp] = tk;
            e[kp] = be;
        }
    }

    template <int W0>
    __device__ __forceinline__ void phase() {
        if constexpr (W0 < NC) {
            constexpr int U0 = W0 * GC / GR;
            const int kend = min((W0 + 1) * GC - 1, ns - 2);
            for (int k = W0 > 0 ? W0 * GC - 1 : 0; k < kend; ++k) {
                const double tk = s_tau[k & 1];
                if (tk != 0.0) {
                    const double* v = vb + (k & 1) * W;
                    double vr[NR], vc[KEEP ? NC : 1], pr[NR];
#pragma unroll
                    for (int u = U0; u < NR; ++u) {
                        vr[u] = v[ti + GR * u];
                        pr[u] = 0.0;
                    }
                    double xn = v[tj + GC * W0];
#pragma unroll
                    for (int w = W0; w < NC; ++w) {
                        const double x = xn;
                        if (w + 1 < NC) xn = v[tj + GC * (w + 1)];
                        if constexpr (KEEP) vc[w] = x;
                        else asm volatile("" ::: "memory");   // one column's read ahead, no more
#pragma unroll
                        for (int u = U0; u < NR; ++u) pr[u] = fma(A[u][w], x, pr[u]);
                    }
                    double pv = 0.0;
#pragma unroll
                    for (int u = U0; u < NR; ++u) {
                        pr[u] = tk * lane_group_sum(pr[u], GC);
                        pv = fma(pr[u], vr[u], pv);
                    }
                    // one value per row group: sum over the row groups of the wave
                    if (GC <= 8) pv += dpp_perm<0x140>(pv);
                    if (GC <= 16) pv = add_xor16(pv);
                    pv = add_xor32(pv);
                    if (tj == 0) {
#pragma unroll
                        for (int u = U0; u < NR; ++u) pb[ti + GR * u] = pr[u];
                    }
                    if ((threadIdx.x & 63) == 0) s_red[threadIdx.x >> 6] = pv;
                    __syncthreads();
                    double sp = 0.0;
#pragma unroll
                    for (int i = 0; i < NW; ++i) sp += s_red[i];
                    const double K = 0.5 * tk * sp;
#pragma unroll
                    for (int u = U0; u < NR; ++u) pr[u] = fma(-K, vr[u], pr[u]);
                    double yn = pb[tj + GC * W0];
                    if constexpr (!KEEP) xn = v[tj + GC * W0];
#pragma unroll
                    for (int w = W0; w < NC; ++w) {
                        const double x = KEEP ? vc[KEEP ? w : 0] : xn, y = yn;
                        if (w + 1 < NC) {
                            yn = pb[tj + GC * (w + 1)];
                            if constexpr (!KEEP) xn = v[tj + GC * (w + 1)];
                        }
                        if constexpr (!KEEP) asm volatile("" ::: "memory");
                        const double wc = fma(-K, x, y);
#pragma unroll
                        for (int u = U0; u < NR; ++u) A[u][w] = fma(-vr[u], wc, fma(-pr[u], x, A[u][w]));
                    }
                }
                if (k + 3 < ns && ti == (k + 1) % GR) pivot<U0, W0>(k + 1);
                __syncthreads();
            }
            phase<W0 + 1>();
        }
    }
};

template <int NR, int NC, int GR, int GC>
__global__ __launch_bounds__(GR * GC) void k_tr_tridiag(TruncArgs a) {
    using T = Tridiag<NR, NC, GR, GC>;
    __shared__ double vbuf[3 * T::W], s_tau[2], s_red[T::NW];
    const TruncLayout L = trunc_layout(a.mp, a.np, a.Dc);
    double* gs = a.scratch + (long long)blockIdx.x * a.ss;
    T t;
    t.Am = gs + L.oA;
    t.e = gs + L.oE;
    t.tau = gs + L.oT;
    t.vb = vbuf;
    t.pb = vbuf + 2 * T::W;
    t.s_tau = s_tau;
    t.s_red = s_red;
    t.ns = L.ns;
    t.lda = L.lda;
    t.ti = threadIdx.x / GC;
    t.tj = threadIdx.x % GC;
    const int ns = L.ns;
    static_assert(GR * GC >= T::W, "a diagonal entry per thread");
    gram_scale<GR * GC>(t.Am, ns, s_red);
#pragma unroll
    for (int u = 0; u < NR; ++u) {
#pragma unroll
        for (int w = 0; w < NC; ++w) {
            const int i = t.ti + GR * u, j = t.tj + GC * w;
            t.A[u][w] = ld_or0(i < ns && j < ns, t.Am, i * L.lda + j);
        }
        asm volatile("" ::: "memory");   // one row's addresses and masks at a time
    }
    __syncthreads();   // the rows of Am are overwritten by the reflectors
    if (ns > 2 && t.ti == 0) t.template pivot<0, 0>(0);
    __syncthreads();
    t.template phase<0>();
#pragma unroll
    for (int u = 0; u < NR; ++u)
#pragma unroll
        for (int w = 0; w < NC; ++w) {
            const int i = t.ti + GR * u, j = t.tj + GC * w;
            if (i == j && i < ns) gs[L.oD + i] = t.A[u][w];
            if (i == ns - 2 && j == ns - 1) t.e[ns - 2] = t.A[u][w];
        }
    if (threadIdx.x == 0) {
        if (ns >= 2) t.tau[ns - 2] = 0.0;
        if (ns >= 1) t.tau[ns - 1] = 0.0;
    }
}

// ---------------------------------------------------------------------------
// tridiagonalisation in memory
// ---------------------------------------------------------------------------
// Orders up to 512, one workgroup of 1024 threads per matrix: panels of 16 steps whose rank-2
// updates are kept as V W^T + W V^T (LDS) and applied to the trailing matrix once per panel
// on the matrix cores, so a step reads the trailing matrix once (p = A v, 16 waves by rows,
// coalesced) and writes nothing.  Bound by that read from L2 or HBM: n^3 / 3 doubles over one
// CU.  Same outputs as k_tr_tridiag.  Order 512, 8 matrices: 79 ms with 256 threads updating the
// matrix in memory at every step, 8.5 ms so.
constexpr int kMemN = 512, kMemB = 16, kMemLd = kMemB + 1;
__global__ __launch_bounds__(1024) void k_tr_tridiag_mem(TruncArgs a) {
    extern __shared__ __align__(16) double msh[];
    double* Vp = msh;                          // kMemN x kMemLd
    double* Wp = Vp + kMemN * kMemLd;
    double* vv = Wp + kMemN * kMemLd;          // current reflector
    double* red = vv + kMemN;                  // 32 partial sums, 32 dot products
    const TruncLayout L = trunc_layout(a.mp, a.np, a.Dc);
    const int n = L.ns, lda = L.lda, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    double* gs = a.scratch + (long long)blockIdx.x * a.ss;
    double *A = gs + L.oA, *d = gs + L.oD, *e = gs + L.oE, *tau = gs + L.oT;
    const auto block_sum = [&](double x) -> double {   // two barriers
        x = lane_group_sum(x, 64);
        if (lane == 0) red[w] = x;
        __syncthreads();
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < 16; ++i) s += red[i];
        __syncthreads();
        return s;
    };
    gram_scale<1024>(A, n, red);
    __syncthreads();
    for (int k0 = 0; k0 < n - 2; k0 += kMemB) {
        const int nb = min(kMemB, n - 2 - k0);
        for (int q = 0; q < nb; ++q) {
            const int k = k0 + q, i = tid;
            // column k of the current matrix: the panel's earlier rank-2 updates applied
            double x = 0.0;
            if (i >= k && i < n) {
                x = A[(long long)k * lda + i];
                for (int s = 0; s < q; ++s)
                    x -= Vp[i * kMemLd + s] * Wp[k * kMemLd + s] + Wp[i * kMemLd + s] * Vp[k * kMemLd + s];
                if (i == k) d[k] = x;
                if (i == k + 1) red[48] = x;
            }
            const double sq = block_sum(i >= k + 2 && i < n ? x * x : 0.0);
            const double al = red[48];
            double tk, be, sc;
            hh_scalars(al, sq, tk, be, sc);
            const double v = i < n ? (i >= k + 2 ? sc * x : (i == k + 1 ? 1.0 : 0.0)) : 0.0;
            if (i < n) {
                vv[i] = v;
                Vp[i * kMemLd + q] = tk != 0.0 ? v : 0.0;
                if (i >= k + 2) A[(long long)k * lda + i] = v;
            }
            if (tid == 0) {
                tau[k] = tk;
                e[k] = be;
            }
            __syncthreads();
            // p = A v over the rows k+1.. of the panel's start matrix, 4 rows of a wave at a time;
            // wave s also forms V_s . v and W_s . v of the earlier columns
            if (tk != 0.0) {
                for (int r0 = k + 1 + 4 * w; r0 < n; r0 += 64) {
                    double s4[4] = {0.0, 0.0, 0.0, 0.0};
                    for (int c = k + 1 + lane; c < n; c += 64) {
                        const double vc = vv[c];
#pragma unroll
                        for (int u = 0; u < 4; ++u)
                            s4[u] = fma(A[(long long)min(r0 + u, n - 1) * lda + c], vc, s4[u]);
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const double s = lane_group_sum(s4[u], 64);
                        if (lane == 0 && r0 + u < n) Wp[(r0 + u) * kMemLd + q] = s;
                    }
                }
                if (w < q) {
                    double gv = 0.0, gw = 0.0;
                    for (int c = k + 1 + lane; c < n; c += 64) {
                        gv = fma(Vp[c * kMemLd + w], vv[c], gv);
                        gw = fma(Wp[c * kMemLd + w], vv[c], gw);
                    }
                    gv = lane_group_sum(gv, 64);
                    gw = lane_group_sum(gw, 64);
                    if (lane == 0) {
                        red[16 + w] = gv;
                        red[32 + w] = gw;
                    }
                }
            }
            __syncthreads();
            double p = 0.0;
            if (tk != 0.0 && i > k && i < n) {
                p = Wp[i * kMemLd + q];
                for (int s = 0; s < q; ++s)
                    p -= Vp[i * kMemLd + s] * red[32 + s] + Wp[i * kMemLd + s] * red[16 + s];
            }
            const double pv = block_sum(p * v);
            if (i < n) Wp[i * kMemLd + q] = tk * fma(-0.5 * tk * pv, v, p);
            __syncthreads();
        }
        // trailing matrix (rows and columns k1..) -= V W^T + W V^T: 16 x 16 tiles, k = 4 s + gq
        const int k1 = k0 + nb, nt = (n - k1 + 15) / 16, li = lane & 15, gq = lane >> 4;
        for (int t = w; t < nt * nt; t += 16) {
            const int r0 = k1 + 16 * (t / nt), c0 = k1 + 16 * (t % nt);
            const int ri = min(r0 + li, n - 1), ci = min(c0 + li, n - 1);
            d4v acc;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = r0 + gq + 4 * r, col = c0 + li;
                acc[r] = ld_or0(row < n && col < n, A, (long long)row * lda + col);
            }
#pragma unroll
            for (int s = 0; s < kMemB / 4; ++s) {
                const int q = 4 * s + gq;
                const double va = q < nb ? -Vp[ri * kMemLd + q] : 0.0, wb = q < nb ? Wp[ci * kMemLd + q] : 0.0;
                const double wa = q < nb ? -Wp[ri * kMemLd + q] : 0.0, vb = q < nb ? Vp[ci * kMemLd + q] : 0.0;
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(va, wb, acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(wa, vb, acc, 0, 0, 0);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = r0 + gq + 4 * r, col = c0 + li;
                if (row < n && col < n) A[(long long)row * lda + col] = acc[r];
            }
        }
        __syncthreads();
    }
    if (tid == 0) {
        const int k = n - 2;   // n > 224 here
        d[k] = A[(long long)k * lda + k];
        d[k + 1] = A[(long long)(k + 1) * lda + k + 1];
        e[k] = A[(long long)k * lda + k + 1];
        tau[k] = tau[k + 1] = 0.0;
    }
}

// ---------------------------------------------------------------------------
// eigenvalues and tridiagonal eigenvectors
// ---------------------------------------------------------------------------
// Eigenvalues (PART & 1) and tridiagonal eigenvectors (PART & 2).  Block = mpb matrices x epb
// eigenvalues x S sub-lanes (bpm blocks cover the tk eigenvalues of a matrix when mpb = 1).
// The S sub-lanes of an eigenvalue (a power of two, so they lie in one wave) evaluate the
// Sturm count at the points of the next log2 S levels of a bisection at once and then follow
// the bisection through them (one point and one level for S = 1); sub-lane 0 then runs the
// inverse iteration.  The points lie on one dyadic grid over [-1, 1], so an eigenvalue does
// not depend on S, nor on the batch from which the launch takes it.
//
// The matrix is scaled by a power of two to a norm in [1/2, 1).  The count comes from the signs
// of the leading principal minors p_i = (d_i - x) p_{i-1} - e_{i-1}^2 p_{i-2}: one dependent
// fma per row and five instructions in all, where the pivots p_i / p_{i-1} cost a reciprocal
// per row; the exponents are brought back every 8 rows (|p| grows by less than 2.5 per row;
// the squared couplings are kept above 1e-36, a change of 1e-18 of the norm, so that two
// consecutive minors cannot both vanish).  The computed minors are those of a matrix within a
// few eps of the norm, as with the pivots.
//
// Both recurrences are bound by instruction issue of their one wave per SIMD: rows are taken
// 8 at a time from arrays padded to whole chunks (padding rows: d = 4, above every x, and
// e = 0), the next chunk's loads in flight during the current one.  The 49 launches of an
// 8x8, D = 4, Dc = 16 amplitude: 6.7 ms with pivots and one row at a time, 3.5 ms so (4096
// samples), 4.2 and 1.5 ms (one sample); order 216, 256 matrices: 550 and 173 us a launch.
// an interval of 2^-51: 4.4e-16 to 8.9e-16 of the norm, which the Rayleigh quotient then leaves
static constexpr int kTriLevels = 52;
__host__ __device__ inline int tri_pad(int n) { return (n + 15) / 16 * 16; }

template <int PART>
__global__ __launch_bounds__(256) void k_eig_tri(TruncArgs a, int S, int mpb, int epb, int bpm) {
    extern __shared__ __align__(16) double tri_lds[];
    const TruncLayout L = trunc_layout(a.mp, a.np, a.Dc);
    const int n = L.ns, tk = L.tk, tid = threadIdx.x, nvl = mpb * epb, nP = tri_pad(n), nd = nP + 17;
    const int grp = blockIdx.x / bpm, part = blockIdx.x % bpm;
    double2* de = reinterpret_cast<double2*>(tri_lds);            // (d_i, e_{i-1}^2), nd per matrix
    double* es = tri_lds + 2LL * mpb * nd;                        // e_i, nP + 16 per matrix
    double* lohi = es + (long long)mpb * (nP + 16);               // Gershgorin bounds, exponent, -
    double2* xl = reinterpret_cast<double2*>(lohi + 4 * mpb);     // (x, 1 / pivot) of every lane
    for (int m2 = tid >> 6; m2 < mpb; m2 += blockDim.x >> 6) {
        const int b2 = grp * mpb + m2, lane = tid & 63;
        const double* g2 = a.scratch + (long long)(b2 < a.batch ? b2 : 0) * a.ss;
        double lo = INFINITY, hi = -INFINITY;
        for (int i = lane; i < n; i += 64) {
            const double dv = g2[L.oD + i];
            const double el = ld_or0(i > 0, g2, L.oE + i - 1), er = ld_or0(i + 1 < n, g2, L.oE + i);
            const double r = fabs(el) + fabs(er);
            lo = fmin(lo, dv - r);
            hi = fmax(hi, dv + r);
        }
        for (int o = 32; o > 0; o >>= 1) {
            lo = fmin(lo, __shfl_xor(lo, o, 64));
            hi = fmax(hi, __shfl_xor(hi, o, 64));
        }
        const double tn = fmax(fabs(lo), fabs(hi));
        const int ex = tn > 0.0 && tn < INFINITY ? __builtin_amdgcn_frexp_exp(tn) : 0;
        for (int i = lane; i < nd; i += 64) {
            const double dv = ld_or0(i < n, g2, L.oD + i), el = ld_or0(i > 0 && i < n, g2, L.oE + i - 1);
            const double sl = __builtin_amdgcn_ldexp(el, -ex);
            de[m2 * nd + i] = make_double2(i < n ? __builtin_amdgcn_ldexp(dv, -ex) : 4.0, fmax(sl * sl, 1e-36));
            if (i < nP + 16)
                es[m2 * (nP + 16) + i] = __builtin_amdgcn_ldexp(ld_or0(i + 1 < n, g2, L.oE + i), -ex);
        }
        if (lane == 0) {
            lohi[4 * m2] = __builtin_amdgcn_ldexp(lo, -ex);
            lohi[4 * m2 + 1] = __builtin_amdgcn_ldexp(hi, -ex);
            lohi[4 * m2 + 2] = (double)ex;
        }
    }
    __syncthreads();
    const int mi = tid / (epb * S), le = tid % (epb * S), l = part * epb + le / S, sub = le % S;
    const int b = grp * mpb + mi;
    if (mi >= mpb || b >= a.batch || l >= tk) return;
    double* gs = a.scratch + (long long)b * a.ss;
    const double2* dm = de + mi * nd;
    const double* e = es + mi * (nP + 16);
    const int ex0 = (int)lohi[4 * mi + 2];
    const double tnorm = fmax(fabs(lohi[4 * mi]), fabs(lohi[4 * mi + 1]));
    double lam;
    if constexpr ((PART & 1) != 0) {
        const int kidx = n - 1 - l;   // l-th largest = kidx-th smallest
        const int lane0 = (tid & 63) - sub;
        const int lev = S == 1 ? 1 : 31 - __clz(S);   // bisection levels per step
        double lo = -1.0;
        for (int done = 0; done < kTriLevels; done += lev) {
            // point `sub` of the 2^lev - 1 interior ones (fewer in the last step): every point is
            // a multiple of 2^-51 and exact
            const int kk = min(lev, kTriLevels - done);
            const double h = __builtin_amdgcn_ldexp(2.0, -(done + kk));
            const double x = fma((double)(sub + 1), h, lo);
            double p0 = 1.0, p1 = dm[0].x - x;
            unsigned cnt = (unsigned)__double2hiint(p1) >> 31;   // eigenvalues below x = sign changes
            double2 q0[8], q1[8];
            const double2* dp = dm + 1;
            const auto load8 = [&](double2 (&q)[8], const double2* src) {
#pragma unroll
                for (int u = 0; u < 8; ++u) q[u] = src[u];
            };
            const auto rows8 = [&](const double2 (&q)[8]) {
                unsigned m = (unsigned)__double2hiint(p1) >> 31;   // the signs, newest in bit 0
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const double p2 = fma(q[u].x - x, p1, -(q[u].y * p0));
                    m = __builtin_amdgcn_alignbit(m, (unsigned)__double2hiint(p2), 31);
                    p0 = p1;
                    p1 = p2;
                }
                cnt += __popc((m ^ (m >> 1)) & 0xffu);
                const int ex = -__builtin_amdgcn_frexp_exp(fmax(fabs(p0), fabs(p1)));
                p0 = __builtin_amdgcn_ldexp(p0, ex);
                p1 = __builtin_amdgcn_ldexp(p1, ex);
            };
            load8(q0, dp);
            for (int i = 1; i < n; i += 16) {
                load8(q1, dp + 8);
                rows8(q0);
                load8(q0, dp + 16);   // past the end of the last chunk: the next matrix's rows or
                rows8(q1);            // the couplings, read and not used
                dp += 16;
            }
            // the descent of a plain bisection through the points: bit j of `above` says that more
            // than kidx eigenvalues lie below point j
            const unsigned long long above = __ballot((int)cnt > kidx) >> lane0;
            int pos = 0;
            for (int s = kk - 1; s >= 0; --s)
                if (!((above >> (pos + (1 << s) - 1)) & 1)) pos += 1 << s;
            lo = fma((double)pos, h, lo);
        }
        if (sub != 0) return;
        lam = lo + __builtin_amdgcn_ldexp(1.0, -kTriLevels);   // the interval's middle
        if constexpr (PART == 1) {
            gs[L.oL + l] = __builtin_amdgcn_ldexp(lam, ex0);
            return;
        }
    } else {
        lam = __builtin_amdgcn_ldexp(gs[L.oL + l], -ex0);
    }
    if constexpr ((PART & 2) != 0) {
        // the lane's iterate with its reciprocal pivots, row i of every lane side by side
        const int xs = nvl;
        double2* xp = xl + mi * epb + (l - part * epb);
        // inverse iteration (T - lam I) x = b with T - lam I = L D L^T, factored once
        const double ptol = fmax(2.220446049250313e-16 * tnorm, 1e-300);
        {
            double pp = 0.0, ep = 0.0;
            for (int i0 = 0; i0 < nP; i0 += 8) {
                double dv[8], ev[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    dv[u] = dm[i0 + u].x - lam;
                    ev[u] = e[i0 + u];
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int i = i0 + u;
                    double q = fma(-(ep * ep), pp, dv[u]);
                    if (fabs(q) < ptol) q = (q < 0.0) ? -ptol : ptol;
                    pp = sturm_rcp(q);
                    ep = ev[u];
                    const double x0 =
                        (double)(hash_u32((unsigned)(l * 7919 + i * 104729 + 17)) & 0xffffff) / 16777216.0 - 0.5;
                    xp[i * xs] = make_double2(i < n ? x0 : 0.0, pp);
                }
            }
        }
        // Per sweep: L y = b upwards (b scaled by sc as it is read), L^T x = D^-1 y downwards
        // with max |x_i|, then the norm of x / max
        double sc = 1.0;
        for (int it = 0; it < 3; ++it) {
            double2 c0[8], c1[8];
            double v0[8], v1[8];
            const auto load8 = [&](double2 (&c)[8], double (&v)[8], int i0) {
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    c[u] = xp[(i0 + u) * xs];
                    v[u] = e[i0 + u];
                }
            };
            double y = 0.0, m = 0.0;   // m: minus the multiplier of the next row
            const auto up8 = [&](const double2 (&c)[8], const double (&v)[8], int i0) {
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    y = fma(m, y, c[u].x * sc);
                    m = -(v[u] * c[u].y);
                    xp[(i0 + u) * xs].x = y;
                }
            };
            load8(c0, v0, 0);
            for (int i0 = 0; i0 < nP; i0 += 16) {
                load8(c1, v1, i0 + 8);
                up8(c0, v0, i0);
                if (i0 + 16 < nP) load8(c0, v0, i0 + 16);
                up8(c1, v1, i0 + 8);
            }
            double xd = 0.0, mx = 0.0;
            const auto down8 = [&](const double2 (&c)[8], const double (&v)[8], int i0) {
#pragma unroll
                for (int u = 7; u >= 0; --u) {
                    xd = fma(-(v[u] * c[u].y), xd, c[u].x * c[u].y);
                    mx = fmax(mx, fabs(xd));
                    xp[(i0 + u) * xs].x = xd;
                }
            };
            load8(c0, v0, nP - 8);
            for (int i0 = nP - 8; i0 > 0; i0 -= 16) {
                load8(c1, v1, i0 - 8);
                down8(c0, v0, i0);
                if (i0 - 16 > 0) load8(c0, v0, i0 - 16);
                down8(c1, v1, i0 - 8);
            }
            const double si = mx > 0.0 ? 1.0 / mx : 1.0;
            double n0 = 0.0, n1 = 0.0;
            for (int i0 = 0; i0 < nP; i0 += 16) {
                double t[16];
#pragma unroll
                for (int u = 0; u < 16; ++u) t[u] = xp[(i0 + u) * xs].x;
#pragma unroll
                for (int u = 0; u < 16; u += 2) {
                    const double t0 = t[u] * si, t1 = t[u + 1] * si;
                    n0 = fma(t0, t0, n0);
                    n1 = fma(t1, t1, n1);
                }
            }
            const double nrm = n0 + n1;
            sc = nrm > 0.0 ? si / sqrt(nrm) : si;
        }
        // the unit vector out, and the eigenvalue from its Rayleigh quotient
        double* xo = gs + L.oX + (long long)l * L.ldx;
        double xq = 0.0, ep = 0.0, rq = 0.0;
        for (int i0 = 0; i0 < nP; i0 += 8) {
            double t[8], dv[8], ev[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                t[u] = xp[(i0 + u) * xs].x * sc;
                dv[u] = dm[i0 + u].x;
                ev[u] = e[i0 + u];
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                rq += t[u] * fma(dv[u], t[u], 2.0 * ep * xq);
                xq = t[u];
                ep = ev[u];
                if (i0 + u < n) xo[i0 + u] = t[u];
            }
        }
        gs[L.oL + l] = __builtin_amdgcn_ldexp(fabs(rq - lam) <= 1e-8 * tnorm ? rq : lam, ex0);
    }
}

// Launch k_eig_tri.  A row of the Sturm count is bound by issue, not by latency, so one wave
// per SIMD saturates the chip and more points per eigenvalue
// only pay while waves are missing: S grows while the lanes fit 1.5 waves per SIMD (steps
// 52 / log2 S, or 52 with one point; S = 2 would be one level on two lanes).  Wide
// matrices are cut into blocks of 256 lanes so that they spread over the CUs, narrow ones
// packed until a wave is full.  The iterates are in LDS, 16 bytes per row and lane (16 lanes of order
// 512: 144 KB).  One launch does both parts where every block
// stays resident with its iterates; a fuller chip takes two, so that the counts, which need
// little LDS, keep all SIMDs busy.
static hipError_t launch_eig_tri(const TruncArgs& a, const TruncLayout& L, size_t cap, hipStream_t st) {
    const int tk = L.tk > 0 ? L.tk : 1, n = L.ns, batch = a.batch;
    struct Shape {
        int S, mpb, epb, bpm, threads;
        long long blocks;
        size_t base, vec;
    };
    const auto shape = [&](int S) {
        Shape t{};
        t.S = S;
        if (tk * S >= 256) {
            t.mpb = 1;
            t.epb = 256 / S;
            t.bpm = (tk + t.epb - 1) / t.epb;
        } else {
            t.epb = tk;
            t.bpm = 1;
            t.mpb = 64 / (tk * S) > 0 ? 64 / (tk * S) : 1;
            if (t.mpb > batch) t.mpb = batch;
        }
        t.threads = (t.mpb * t.epb * S + 63) / 64 * 64;
        t.blocks = (long long)((batch + t.mpb - 1) / t.mpb) * t.bpm;
        t.base = (size_t)t.mpb * (2 * (tri_pad(n) + 17) + tri_pad(n) + 16 + 4) * sizeof(double) + 256;
        t.vec = (size_t)t.mpb * t.epb * tri_pad(n) * 2 * sizeof(double);
        return t;
    };
    int S = 1;
    for (int s = 4; s <= 32; s *= 2)
        if ((long long)batch * tk * s <= 98304) S = s;
    const Shape v = shape(S);
#define TRI(PART_, sh, bytes_)                                                                              \
    hipLaunchKernelGGL((k_eig_tri<PART_>), dim3((unsigned)sh.blocks), dim3(sh.threads), (bytes_), st, a, \
                       sh.S, sh.mpb, sh.epb, sh.bpm)
    const size_t both = v.base + v.vec;
    if (both <= cap && (v.blocks + 255) / 256 <= (long long)(cap / both)) {
        TRI(3, v, both);
        return hipGetLastError();
    }
    TRI(1, v, v.base);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    Shape w = shape(1);
    while (w.mpb > 1 && w.base + w.vec > cap) {   // fewer matrices, then fewer lanes of one
        const int half = w.mpb / 2;
        w.base = (w.base - 256) / w.mpb * half + 256;
        w.vec = w.vec / w.mpb * half;
        w.mpb = half;
        w.threads = (w.mpb * w.epb + 63) / 64 * 64;
        w.blocks = (batch + w.mpb - 1) / w.mpb;
    }
    if (w.base + w.vec > cap) {
        while (w.epb > 16 && w.base + w.vec > cap) {
            w.epb = (w.epb + 1) / 2;
            w.vec = (size_t)w.epb * tri_pad(n) * 2 * sizeof(double);
        }
        w.bpm = (tk + w.epb - 1) / w.epb;
        w.threads = (w.epb + 63) / 64 * 64;
        w.blocks = (long long)batch * w.bpm;
    }
    if (w.base + w.vec > cap) return hipErrorInvalidValue;
    TRI(2, w, w.base + w.vec);
#undef TRI
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// kept subspace, new tensor, carried right part
// ---------------------------------------------------------------------------
// out(x, k) = sum_y Mat(x, y) B(y, k) with Mat(x, y) = Mat[x ld + y] (ROWS) or Mat[y ld + x],
// B(y, k) = B[k ldb + y], the result at out + x out_x + k out_k, on the matrix cores.  Wave w takes
// the row tiles w, w + NW, ... and all NC column tiles.  Step s of a chunk of 16 y takes
// y = 4 gq + s, so a lane reads four consecutive y.
template <int NW, int NC, bool ROWS>
__device__ __forceinline__ void mat_product(const double* Mat, int ld, int nx, int ny, int tk, const double* B,
                                            int ldb, double* out, long long out_x, long long out_k) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, li = lane & 15, gq = lane >> 4;
    for (int x0 = 16 * w; x0 < nx; x0 += 16 * NW) {
        const int x = x0 + li;
        d4v acc[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) acc[c] = d4v{0.0, 0.0, 0.0, 0.0};
        for (int y0 = 0; y0 < ny; y0 += 32) {
            double av[8], bv[8][NC];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int y = y0 + 16 * (u >> 2) + 4 * gq + (u & 3);
                const bool ok = y < ny;
                av[u] = ld_or0(ok && x < nx, Mat, ROWS ? (long long)x * ld + y : (long long)y * ld + x);
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    const int k = 16 * c + li;
                    bv[u][c] = ld_or0(ok && k < tk, B, (long long)k * ldb + y);
                }
            }
#pragma unroll
            for (int u = 0; u < 8; ++u)
#pragma unroll
                for (int c = 0; c < NC; ++c)
                    acc[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[u], bv[u][c], acc[c], 0, 0, 0);
        }
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int xr = x0 + gq + 4 * r, k = 16 * c + li;
                if (xr < nx && k < tk) out[xr * out_x + k * out_k] = acc[c][r];
            }
    }
}

// Orthonormal basis of the m x tk block X (column-major) in place.  Columns are scaled by a power
// of two as they are loaded, which changes no subspace and keeps their squared norms in range.
template <int NW, int SL, int RPL>
__device__ __forceinline__ void block_orth(double* X, int m, int tk, double (*vbuf)[64 * RPL], double* tau) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    double a[SL][RPL];
#pragma unroll
    for (int s = 0; s < SL; ++s) {
        const int j = s * NW + w;
        double mx = 0.0;
#pragma unroll
        for (int r = 0; r < RPL; ++r) {
            const int i = lane + 64 * r;
            a[s][r] = (j < tk && i < m) ? X[(long long)j * m + i] : 0.0;
            mx = fmax(mx, fabs(a[s][r]));
        }
        for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o, 64));
        const int ex = mx > 0.0 ? -__builtin_amdgcn_frexp_exp(mx) : 0;
#pragma unroll
        for (int r = 0; r < RPL; ++r) a[s][r] = __builtin_amdgcn_ldexp(a[s][r], ex);
    }
    thinq_factor<NW, SL, RPL>(a, tk, vbuf, tau);
    __syncthreads();
    thinq_form<NW, SL, RPL>(a, tk, vbuf, tau);
#pragma unroll
    for (int s = 0; s < SL; ++s) {
        const int j = s * NW + w;
#pragma unroll
        for (int r = 0; r < RPL; ++r) {
            const int i = lane + 64 * r;
            if (j < tk && i < m) X[(long long)j * m + i] = a[s][r];
        }
    }
}

// X <- H_0 ... H_{ns-3} X (the reflectors of the tridiagonalisation, row k of Am beyond k+1, unit
// entry at k+1) in compact WY blocks of 16, on the matrix cores.  X (ns x tk at Xg, ld ldx) is
// held in the MFMA accumulator layout, wave w owning the row tiles w, w + NW, ...: register r of
// a tile is then also the k-step operand whose four rows are gq + 4 r, so V^T X and V^T V read it
// as it is.  Per block: W = V^T X (partial sums of the waves, multiplied by T before they are
// added), then X -= V W; two barriers.  Tl: LDS, 256 doubles per block of reflectors; Wl: LDS,
// (NW + 1) 16 x 16 NC doubles.  The result goes to out (column-major, ld ldo).
template <int NW, int NC, int RT>
__device__ __forceinline__ void back_transform(const double* Xg, int ldx, const double* Am, int lda,
                                               const double* tau, int ns, int tk, double* out, int ldo, double* Tl,
                                               double* Wl) {
    constexpr int CW = 16 * NC;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, li = lane & 15, gq = lane >> 4;
    const int nr = ns - 2, nblk = nr > 0 ? (nr + 15) / 16 : 0;
    const auto vval = [&](int k, int j) -> double {
        const bool in = k < nr && j > k + 1 && j < ns;
        const double x = ld_or0(in, Am, (long long)k * lda + j);
        return (k < nr && j == k + 1) ? 1.0 : x;
    };
    // T of every block: V^T V, then T_jj = tau_j, T[0:j, j] = -tau_j T[0:j, 0:j] (V^T V)[0:j, j];
    // row i of T needs only its own earlier entries
    for (int b = w; b < nblk; b += NW) {
        const int k0 = 16 * b;
        d4v acc = {0.0, 0.0, 0.0, 0.0};
        for (int r0 = k0 / 16 * 16; r0 < ns; r0 += 16) {
            double v[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = vval(k0 + li, r0 + gq + 4 * r);
#pragma unroll
            for (int r = 0; r < 4; ++r) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(v[r], v[r], acc, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int q = gq + 4 * r;   // the diagonal, not needed, takes tau
            Tl[b * 256 + q * 16 + li] = q != li ? acc[r] : (k0 + q < nr ? tau[k0 + q] : 0.0);
        }
    }
    __syncthreads();
    double row[16];
    for (int b0 = 0; b0 < nblk; b0 += NW) {
        const int b = b0 + w;
        if (b < nblk && lane < 16) {
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const double* g = Tl + b * 256 + j;
                double s = 0.0;
#pragma unroll
                for (int q = 0; q < 16; ++q)
                    if (q < j) s = fma(row[q], g[q * 16], s);   // row[q] = 0 for q < lane
                const double tj = g[j * 16];
                row[j] = j < lane ? 0.0 : (j == lane ? tj : -tj * s);
                asm volatile("" : "+v"(row[j])::"memory");   // one column's LDS reads at a time
            }
        }
        __syncthreads();
        if (b < nblk && lane < 16)
#pragma unroll
            for (int j = 0; j < 16; ++j) Tl[b * 256 + lane * 16 + j] = row[j];
        __syncthreads();
    }
    d4v x[RT][NC];
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = 16 * (w + NW * t) + gq + 4 * r, k = 16 * c + li;
                x[t][c][r] = ld_or0(i < ns && k < tk, Xg, (long long)k * ldx + i);
            }
    double* red = Wl;
    double* Ws = Wl + NW * 16 * CW;
    for (int b = nblk - 1; b >= 0; --b) {
        const int k0 = 16 * b;
        d4v wp[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) wp[c] = d4v{0.0, 0.0, 0.0, 0.0};
        double uv[RT][4];   // V of the own rows for the update, loaded early
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            const int r0 = 16 * (w + NW * t);
            const bool live = r0 < ns && r0 + 15 > k0;
            if (live) {
                double v[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] = vval(k0 + li, r0 + gq + 4 * r);
#pragma unroll
                for (int r = 0; r < 4; ++r) uv[t][r] = -vval(k0 + 4 * r + gq, r0 + li);
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int c = 0; c < NC; ++c)
                        wp[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(v[r], x[t][c][r], wp[c], 0, 0, 0);
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r) uv[t][r] = 0.0;
            }
        }
        double ta[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) ta[r] = Tl[b * 256 + li * 16 + gq + 4 * r];
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            d4v q = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int r = 0; r < 4; ++r) q = __builtin_amdgcn_mfma_f64_16x16x4f64(ta[r], wp[c][r], q, 0, 0, 0);
#pragma unroll
            for (int r = 0; r < 4; ++r) red[(w * 16 + gq + 4 * r) * CW + 16 * c + li] = q[r];
        }
        __syncthreads();
        for (int i = tid; i < 16 * CW; i += 64 * NW) {
            double s = 0.0;
#pragma unroll
            for (int u = 0; u < NW; ++u) s += red[u * 16 * CW + i];
            Ws[i] = s;
        }
        __syncthreads();
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const double bw = Ws[(4 * s + gq) * CW + 16 * c + li];
#pragma unroll
                for (int t = 0; t < RT; ++t)
                    x[t][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(uv[t][s], bw, x[t][c], 0, 0, 0);
            }
    }
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = 16 * (w + NW * t) + gq + 4 * r, k = 16 * c + li;
                if (i < ns && k < tk) out[(long long)k * ldo + i] = x[t][c][r];
            }
}

// One workgroup per matrix, mp, np <= 64 RPL and tk <= NW SL:
//   the tridiagonal eigenvectors orthonormalised (thin Householder QR, thinq.h) and carried
//   back to the Gram matrix's;
//   order mp (left singular vectors U): V = orth(M^T U);
//   where the Gram route is too coarse, one step of orthogonal iteration on M itself,
//   V <- orth(M^T orth(M V)), every product acting on orthonormal vectors: the Gram eigenvectors
//   locate the kept subspace only to about eps lambda_1 / (lambda_t - lambda_{t+1}), this to
//   eps sigma_1 / (sigma_t - sigma_{t+1}).  That is where a kept eigenvalue is below 1e-6 of the
//   largest, and always for orders above 224, where the step is cheap beside the rest and the
//   Gram route alone left ln|W| of a 24 x 24, D = 8 state ten times the oracle's rounding noise
//   away;
//   H = F V.
// Bound by the chain of reflector steps, 2 tk per orthonormalisation and about 0.9 us each: one of
// them for order np, two for order mp, and two more with refinement (2, 4, 6 or 8 tk steps);
// the blocks pass between the phases through the scratch (L2).  Order 216, tk = 36, 256 matrices
// without refinement: 217 us, where Gram-Schmidt and one reflector at a time from memory took
// 607 us and left the carried factor to be formed; 48 matrices with it: 385 us against 543 us
// and 4.3 ms for a refinement with its blocks in memory.
template <int NW, int SL, int RPL>
__global__ __launch_bounds__(NW * 64, SL * RPL <= 8 ? 4 : 2) void k_tr_vec(TruncArgs a) {
    constexpr int NC = (NW * SL + 15) / 16, RT = (4 * RPL + NW - 1) / NW;
    extern __shared__ __align__(16) double vsh[];   // back_transform: Wl, then Tl
    __shared__ double vbuf[2][64 * RPL];
    __shared__ double htau[NW * SL];
    const TruncLayout L = trunc_layout(a.mp, a.np, a.Dc);
    const int b = blockIdx.x, mp = a.mp, np = a.np, tk = L.tk, ns = L.ns;
    double* gs = a.scratch + (long long)b * a.ss;
    const double* M = gs + L.oM;
    double *X = gs + L.oX, *Y = gs + L.oY;
    double* V = a.newU + (long long)b * a.us;
    block_orth<NW, SL, RPL>(X, ns, tk, vbuf, htau);
    __syncthreads();
    back_transform<NW, NC, RT>(X, L.ldx, gs + L.oA, L.lda, gs + L.oT, ns, tk, L.gram_right ? V : Y,
                               L.gram_right ? np : mp, vsh + (NW + 1) * 256 * NC, vsh);
    __syncthreads();
    if (!L.gram_right) {
        mat_product<NW, NC, false>(M, np, np, mp, tk, Y, mp, V, 1, np);
        __syncthreads();
        block_orth<NW, SL, RPL>(V, np, tk, vbuf, htau);
        __syncthreads();
    }
    const double l0 = gs[L.oL], lt = gs[L.oL + tk - 1];
    if (l0 > 0.0 && (lt < 1e-6 * l0 || ns > 224)) {
        mat_product<NW, NC, true>(M, np, mp, np, tk, V, np, Y, 1, mp);
        __syncthreads();
        block_orth<NW, SL, RPL>(Y, mp, tk, vbuf, htau);
        __syncthreads();
        mat_product<NW, NC, false>(M, np, np, mp, tk, Y, mp, V, 1, np);
        __syncthreads();
        block_orth<NW, SL, RPL>(V, np, tk, vbuf, htau);
        __syncthreads();
    }
    mat_product<NW, NC, true>(a.F + (long long)b * a.fs, np, a.nf, np, tk, V, np, a.H + (long long)b * a.hs, tk, 1);
}

// The smallest blocking of k_tr_vec that holds the blocks; false when none does.  NW waves of SL
// columns and 64 RPL rows: one wave per SIMD up to 16 columns (a second one only adds to a step),
// two for more; blocks of 64 rows that hold nothing cost every step.  (8, 5, 4) is there because 33 to 40
// columns of up to 256 rows would else run in twice the registers and twice the rows (8, 8, 8):
// order 216, 36 columns, truncation class of a 12x12 evaluation (48 samples) 170 ms with it, 207 ms
// without; 16x16 amplitudes (256 samples) 164 and 187 ms.
template <class Fn>
bool vec_blocking(int m, int t, Fn&& fn) {
#define VB(NW_, SL_, RPL_) \
    if (m <= 64 * RPL_ && t <= NW_ * SL_) { fn.template operator()<NW_, SL_, RPL_>(); return true; }
    VB(4, 4, 1)
    VB(4, 4, 2)
    VB(8, 4, 2)
    VB(8, 5, 4)
    VB(8, 4, 8)
    VB(8, 8, 8)
#undef VB
    return false;
}

struct VecFits {
    template <int NW, int SL, int RPL> void operator()() const {}
};
struct VecLaunch {
    const TruncArgs& a;
    int ns;
    hipStream_t st;
    template <int NW, int SL, int RPL> void operator()() const {
        const int nblk = ns > 2 ? (ns - 2 + 15) / 16 : 0;
        const size_t bytes = ((size_t)(NW + 1) * 256 * ((NW * SL + 15) / 16) + 256 * (size_t)nblk) * sizeof(double);
        hipLaunchKernelGGL((k_tr_vec<NW, SL, RPL>), dim3(a.batch), dim3(64 * NW), bytes, st, a);
    }
};

}  // namespace

bool trunc_fits(int mp, int np, int Dc) {
    const TruncLayout L = trunc_layout(mp, np, Dc);
    return L.ns <= kMemN && vec_blocking(mp > np ? mp : np, L.tk, VecFits{});
}

size_t trunc_scratch_doubles(int mp, int np, int Dc) { return (size_t)trunc_layout(mp, np, Dc).total; }

hipError_t launch_trunc(const TruncArgs& a, hipStream_t st) {
    if (a.batch <= 0) return hipSuccess;
    if (!trunc_fits(a.mp, a.np, a.Dc)) return hipErrorInvalidValue;
    const TruncLayout L = trunc_layout(a.mp, a.np, a.Dc);
    const size_t cap = get_lds_cap() - 1024;
    // Gram matrix (symmetric, so the stored rows are its columns too)
    GemmArgs g{};
    const Idx2 one{1 << 30, 0, 1}, ld{1 << 30, 0, (long long)a.np};
    g.M = g.N = L.ns;
    g.K = L.gram_right ? a.mp : a.np;
    g.batch = a.batch;
    g.am = L.gram_right ? one : ld;
    g.ak = L.gram_right ? ld : one;
    g.bk = g.ak;
    g.bn = g.am;
    g.cm = Idx2{1 << 30, 0, (long long)L.lda};
    g.cn = one;
    g.a_bs = g.b_bs = g.c_bs = a.ss;
    g.A = g.B = a.scratch + L.oM;
    g.C = a.scratch + L.oA;
    g.alpha = 1.0;
    hipError_t e = launch_mgemm(g, Arith::F64, st, 0);
    if (e != hipSuccess) return e;
    const dim3 grid(a.batch);
    if (L.ns <= 16) hipLaunchKernelGGL((k_tr_tridiag<2, 2, 8, 8>), grid, dim3(64), 0, st, a);
    else if (L.ns <= 32) hipLaunchKernelGGL((k_tr_tridiag<4, 4, 8, 8>), grid, dim3(64), 0, st, a);
    else if (L.ns <= 64) hipLaunchKernelGGL((k_tr_tridiag<8, 8, 8, 8>), grid, dim3(64), 0, st, a);
    else if (L.ns <= 128) hipLaunchKernelGGL((k_tr_tridiag<4, 8, 32, 16>), grid, dim3(512), 0, st, a);
    else if (L.ns <= 224) hipLaunchKernelGGL((k_tr_tridiag<7, 14, 32, 16>), grid, dim3(512), 0, st, a);
    else
        hipLaunchKernelGGL(k_tr_tridiag_mem, grid, dim3(1024), (2 * kMemN * kMemLd + kMemN + 64) * sizeof(double), st, a);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    e = launch_eig_tri(a, L, cap, st);
    if (e != hipSuccess) return e;
    vec_blocking(a.mp > a.np ? a.mp : a.np, L.tk, VecLaunch{a, L.ns, st});
    return hipGetLastError();
}

}  // namespace peps
