// Fused single- and two-row sandwich steps in float64 (Sec. 3, Eq. (4)): one launch in
// place of three or four batched GEMMs whose temporaries (bond^2 legs^3 per sample) make
// the round trip through memory, and, where one workgroup holds a whole sample, of the
// rescaling of the result too.
//
// Both directions are the same chain over renamed legs (the launcher passes strides):
//   T1[b,b',g,u,f']  = sum_f      X[f,b,b',g]  E1[f,u,f']
//   T2[b',g,f',a,m]  = sum_{b,u}  T1 A[b,u,a,m]
//   T3[g,f',a,a',q]  = sum_{b',m} T2 B[b',m,a',q]          (two-row step only)
//   Y[f',a,a',g']    = sum_{g,q}  T3 E2[g,q,g']
// f' stays free to the end, so a workgroup takes NF values of it and keeps that slice of
// the temporary in LDS, where T2 and T3 replace their input in place: a wave reads the
// whole K of its 16 rows before it writes them, and the rows of T3, (f',g,a), are
// disjoint sets of entries.  Rows of T2 (f',g,b') are RS doubles apart, RS odd for the LDS
// banks.  All four products run on 16x16x4 MFMAs, A operands from memory (T1) or LDS, B
// operands from memory through L1, held in registers for T2 and T3.  Every output sums in
// the k order of its GEMM, so the results are equal to those of the GEMM form bit for bit.
//
// Bound by latency at small samples, by LDS and latency at D = 4 (8x8, 4096 samples, 99 us a step: 1.5 TB/s,
// matrix cores 15 % busy).  A step, mean over an evaluation: 4x4 D = 2, 256 samples, three or four
// launches of 3.4 us and a rescaling of 3.2 -> 6.0 us; 8x8 D = 4, bond 16, 512 samples, launches of 8 to 13 us each -> 19 us.
#include <algorithm>

#include "common.h"
#include "kernels.h"
#include "mfma_ops.h"

namespace peps {

namespace {

constexpr int kStepNT = 256, kSite = 16, KS = kSite / 4;   // threads; K and N of a site product
// LDS of a workgroup: four of them on a compute unit
constexpr long long kStepLds = 40 * 1024;

// division by a launch constant: i / d by multiply-high (exact while i d < 2^32)
struct Div {
    unsigned d, magic;
};
Div make_div(int d) { return Div{(unsigned)d, d > 1 ? (unsigned)((1LL << 32) / d + 1) : 0u}; }
__device__ __forceinline__ int div_of(int i, const Div& x) {
    return x.magic ? (int)__umulhi((unsigned)i, x.magic) : i;
}

struct StepP {
    StepArgs a;
    int nf, fblocks, hm, rs, dm;      // f' values and blocks of a workgroup; LDS row shape
    Div dg, du, dgr, dh1, dmid, da1, dk4;
    Div din4;                         // stage 4 k: inner size and strides (LDS, E2)
    int aso, asi, bso, bsi;
};

__device__ __forceinline__ mf64x4 zero4() { return mf64x4{0.0, 0.0, 0.0, 0.0}; }

// B operand of a site product, all k steps: lane (li, gq) of step s holds
// S(min(k, K - 1), li), k = 4 s + gq, k = (ko, ki) and n = (no, ni) with their strides
__device__ __forceinline__ void site_frag(double (&f)[KS], const double* S, int K, int N, const Div& dk, int sko,
                                          int ski, const Div& dn, int sno, int sni, int li, int gq) {
    const int n = min(li, N - 1), no = div_of(n, dn), on = no * sno + (n - no * (int)dn.d) * sni;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        const int k = 4 * s + gq, kk = min(k, K - 1), ko = div_of(kk, dk);
        const int ok = ko * sko + (kk - ko * (int)dk.d) * ski;
        f[s] = S[ok + on];
    }
}

// E2 operand of k steps s0 .. s0 + 31 of the last product (past K: its last entry)
__device__ __forceinline__ void e2_load(double (&v)[8], const double* er, int s0, int K, const StepP& p, int gq) {
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        const int k = min(s0 + 4 * s + gq, K - 1), ko = div_of(k, p.din4);
        v[s] = er[ko * p.bso + (k - ko * (int)p.din4.d) * p.bsi];
    }
}

__global__ __launch_bounds__(kStepNT) void k_step64(StepP p) {
    extern __shared__ __align__(16) double W[];
    constexpr int NW = kStepNT / 64;
    __shared__ double red[NW];
    const StepArgs& a = p.a;
    const int b = blockIdx.x / p.fblocks, f0 = (blockIdx.x % p.fblocks) * p.nf;
    if (b >= a.batch) return;
    if (a.skip && a.skip[(long long)b * a.skip_bs] == 0) return;
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, gq = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nf = min(p.nf, a.F1 - f0);
    const int G = a.G, H = a.H, H1 = a.H1, hb = a.pair ? H : 1, hb1 = a.pair ? H1 : 1, hm = p.hm, RS = p.rs;
    const double* X = a.X + (long long)b * a.xs;
    const double* E1 = a.E1 + (long long)b * a.e1s;
    const double* E2 = a.E2 + (long long)b * a.e2s;
    const double* SA = a.SA + (long long)((a.selA[(long long)b * a.sel_bs] ^ a.flipA) & 1) * a.slice;
    const double* SB = a.SB + (long long)((a.selB[(long long)b * a.sel_bs] ^ a.flipB) & 1) * a.slice;
    double* Y = a.Y + (long long)b * a.ys;

    // the site operands and the first of E2 are loaded ahead of their stages
    double frA[KS], frB[KS], e2[8];
    site_frag(frA, SA, H * a.Du, H1 * a.Dm, p.du, a.sak[0], a.sak[1], p.dk4, a.san[0], a.san[1], li, gq);
    site_frag(frB, SB, H * a.Dm, H1 * a.Dq, p.dk4, a.sbk[0], a.sbk[1], p.da1, a.sbn[0], a.sbn[1], li, gq);
    const int M4 = nf * H1 * hb1, N4 = a.G1, K4 = G * a.Dq, mt4 = (M4 + 15) / 16, nt4 = (N4 + 15) / 16;
    auto e2_col = [&](int t) { return E2 + (long long)min(16 * (t / mt4) + li, N4 - 1) * a.e2g1; };
    if (w < mt4 * nt4) e2_load(e2, e2_col(w), 0, K4, p, gq);

    {   // stage 1: rows m = (b, b', g), columns n = (f', u)
        const int M = H * hb * G, N = nf * a.Du, mt = (M + 15) / 16, nt = (N + 15) / 16, K = a.F;
        for (int t = w; t < mt * nt; t += NW) {
            const int nb = t / mt, mb = t - nb * mt;
            const int m = min(16 * mb + li, M - 1), n = min(16 * nb + li, N - 1);
            const int mi = div_of(m, p.dg), g = m - mi * G, bb = div_of(mi, p.dmid), b2 = mi - bb * hb;
            const int fp = div_of(n, p.du), u = n - fp * a.Du;
            const double* xa = X + (bb * a.xb + b2 * a.xb2 + g * a.xg);
            const double* xe = E1 + (u * a.e1u + (f0 + fp) * a.e1f1);
            mf64x4 acc = zero4();
            for (int s0 = 0; s0 < K; s0 += 16) {
                double va[4], ve[4];
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const int k = s0 + 4 * s + gq, kk = min(k, K - 1);
                    va[s] = xa[(long long)kk * a.xf];
                    ve[s] = xe[(long long)kk * a.e1f];
                }
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    if (s0 + 4 * s >= K) break;
                    const bool in = s0 + 4 * s + gq < K;
                    acc = mfma<Arith::F64>(in ? va[s] : 0.0, in ? ve[s] : 0.0, acc);
                }
            }
            if (16 * nb + li < N) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int mo = 16 * mb + gq + 4 * r;
                    const int q = div_of(mo, p.dg), go = mo - q * G, bo = div_of(q, p.dmid), b2o = q - bo * hb;
                    if (mo < M) W[((fp * G + go) * hm + b2o) * RS + bo * a.Du + u] = acc[r];
                }
            }
        }
    }
    __syncthreads();
    {   // stage 2, in place: rows (f', g, b'), k = (b, u), columns (a, m)
        const int R = nf * G * hb, K = H * a.Du, N = H1 * a.Dm;
        const int no = div_of(li, p.dk4), col = li < N ? no * p.dm + (li - no * a.Dm) : -1;
        for (int t = w; t < (R + 15) / 16; t += NW) {
            const int r0 = min(16 * t + li, R - 1), q0 = div_of(r0, p.dmid);
            const double* wr = W + (q0 * hm + (r0 - q0 * hb)) * RS;
            mf64x4 acc = zero4();
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                if (4 * s >= K) break;
                const int k = 4 * s + gq;
                const double v = wr[min(k, K - 1)], av = k < K ? v : 0.0;
                acc = mfma<Arith::F64>(av, k < K ? frA[s] : 0.0, acc);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int ro = 16 * t + gq + 4 * r, q = div_of(ro, p.dmid);
                double* wo = W + (q * hm + (ro - q * hb)) * RS;
                if (ro < R && col >= 0) wo[col] = acc[r];
            }
        }
    }
    if (a.pair) {   // stage 3, in place: rows (f', g, a), k = (b', m), columns (a', q)
        __syncthreads();
        const int R = nf * G * H1, K = H * a.Dm, N = H1 * a.Dq;
        const int no = div_of(li, p.da1), col = li < N ? no * RS + (li - no * a.Dq) : -1;
        for (int t = w; t < (R + 15) / 16; t += NW) {
            const int r0 = min(16 * t + li, R - 1), q0 = div_of(r0, p.dh1);
            const double* wr = W + q0 * hm * RS + (r0 - q0 * H1) * p.dm;
            mf64x4 acc = zero4();
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                if (4 * s >= K) break;
                const int k = 4 * s + gq, kk = min(k, K - 1), ko = div_of(kk, p.dk4);
                const double v = wr[ko * RS + (kk - ko * a.Dm)], av = k < K ? v : 0.0;
                acc = mfma<Arith::F64>(av, k < K ? frB[s] : 0.0, acc);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int ro = 16 * t + gq + 4 * r, q = div_of(ro, p.dh1);
                double* wo = W + q * hm * RS + (ro - q * H1) * p.dm;
                if (ro < R && col >= 0) wo[col] = acc[r];
            }
        }
    }
    __syncthreads();
    // stage 4: rows (f', a, a'), k = (g, q) in the GEMM's order, columns g'
    const int M = M4, N = N4, mt = mt4, nt = nt4;
    constexpr int TMAX = 2;   // output tiles a wave holds for the rescaling
    mf64x4 keep[TMAX];
    double mx = 0.0;
    auto store = [&](int t, const mf64x4& acc, double scale) {
        const int nb = t / mt, mb = t - nb * mt, n = 16 * nb + li;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = 16 * mb + gq + 4 * r, q = div_of(m, p.dgr), a2 = m - q * hb1, fp = div_of(q, p.dh1),
                      a1 = q - fp * H1;
            if (m < M && n < N)
                Y[(long long)(f0 + fp) * a.yf + a1 * a.ya + a2 * a.ya2 + (long long)n * a.yg] = acc[r] * scale;
        }
    };
#pragma unroll
    for (int it = 0; it < TMAX; ++it) keep[it] = zero4();
    auto tile = [&](int t) -> mf64x4 {
        const int nb = t / mt, mb = t - nb * mt;
        const int m = min(16 * mb + li, M - 1), n = min(16 * nb + li, N - 1);
        const int q = div_of(m, p.dgr), a2 = m - q * hb1, fp = div_of(q, p.dh1), a1 = q - fp * H1;
        const double* wr = W + (fp * G * hm + a2) * RS + a1 * p.dm;
        const double* er = e2_col(t);
        mf64x4 acc = zero4();
        for (int s0 = 0; s0 < K4; s0 += 32) {
            double va[8], ve[8];
#pragma unroll
            for (int s = 0; s < 8; ++s) ve[s] = e2[s];
            if (t != w || s0) e2_load(ve, er, s0, K4, p, gq);
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                const int k = min(s0 + 4 * s + gq, K4 - 1), ko = div_of(k, p.din4);
                va[s] = wr[ko * p.aso + (k - ko * (int)p.din4.d) * p.asi];
            }
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                if (s0 + 4 * s >= K4) break;
                const bool in = s0 + 4 * s + gq < K4;
                acc = mfma<Arith::F64>(in ? va[s] : 0.0, in ? ve[s] : 0.0, acc);
            }
        }
        return acc;
    };
    if (!a.lout) {
        for (int t = w; t < mt * nt; t += NW) store(t, tile(t), 1.0);
        return;
    }
    // rescaling (one workgroup per sample): the largest |entry|, as the separate kernel does it
#pragma unroll
    for (int it = 0; it < TMAX; ++it) {
        const int t = w + it * NW;
        if (t >= mt * nt) continue;
        keep[it] = tile(t);
        const int nb = t / mt, mb = t - nb * mt;
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (16 * mb + gq + 4 * r < M && 16 * nb + li < N) mx = fmax(mx, fabs(keep[it][r]));
    }
    for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o, 64));
    if (lane == 0) red[w] = mx;
    __syncthreads();
    mx = red[0];
#pragma unroll
    for (int i = 1; i < NW; ++i) mx = fmax(mx, red[i]);
    const bool ok = mx > 0.0 && isfinite(mx);
    if (tid == 0) a.lout[b] = (a.lin ? a.lin[b] : 0.0) + (ok ? log(mx) : 0.0);
    const double inv = ok ? 1.0 / mx : 1.0;
#pragma unroll
    for (int it = 0; it < TMAX; ++it)
        if (w + it * NW < mt * nt) store(w + it * NW, keep[it], inv);
}

struct StepPlan {
    int nf, hm, rs, dm;
    long long lds;
    bool whole;   // one workgroup per sample
};

// Site products of K and N up to 16, one MFMA tile of columns and four k steps held in registers:
// legs up to 4.  Wider ones (D = 6: 36 x 36, 140 KB of LDS, one workgroup per compute unit) ran slower
// than their products (12x12 evaluation 412 -> 451 ms).  A sample of at most 32 KB goes to one
// workgroup, which then rescales it; else as many f' as fill the 16 columns of the first product.
bool plan_of(const StepArgs& a, StepPlan& s) {
    const int hb = a.pair ? a.H : 1, hb1 = a.pair ? a.H1 : 1, dq = a.pair ? a.Dq : a.Dm;
    const int k2 = std::max(a.H * a.Du, a.pair ? a.H * a.Dm : 1), n2 = std::max(a.H1 * a.Dm, a.pair ? a.H1 * a.Dq : 1);
    if (k2 > kSite || n2 > kSite) return false;
    s.hm = std::max(hb, hb1);
    s.dm = std::max(a.Dm, dq);
    s.rs = std::max(a.H * a.Du, a.H1 * s.dm) | 1;
    const long long per = 8LL * a.G * s.hm * s.rs;   // LDS of one f'
    const int tiles = ((a.F1 * a.H1 * hb1 + 15) / 16) * ((a.G1 + 15) / 16);
    s.whole = per * a.F1 <= 32 * 1024 && tiles <= 8;
    s.nf = s.whole ? a.F1 : (int)std::min<long long>(std::max(1, 16 / a.Du), kStepLds / per);
    s.nf = std::min(s.nf, a.F1);
    if (s.nf < 1) return false;
    s.lds = per * s.nf;
    return true;
}

}  // namespace

bool step64_fits(const StepArgs& a) {
    StepPlan s;
    return plan_of(a, s);
}
bool step64_rescales(const StepArgs& a) {
    StepPlan s;
    return plan_of(a, s) && s.whole;
}

hipError_t launch_step64(const StepArgs& a0, hipStream_t st) {
    StepPlan s;
    if (a0.batch <= 0) return hipSuccess;
    if (!plan_of(a0, s)) return hipErrorInvalidValue;
    StepP p;
    p.a = a0;
    if (!p.a.pair) p.a.Dq = p.a.Dm;
    if (!s.whole) p.a.lout = nullptr;
    const StepArgs& a = p.a;
    p.nf = s.nf;
    p.fblocks = (a.F1 + s.nf - 1) / s.nf;
    p.hm = s.hm; p.rs = s.rs; p.dm = s.dm;
    p.dg = make_div(a.G);
    p.du = make_div(a.Du);
    p.dmid = make_div(a.pair ? a.H : 1);
    p.dgr = make_div(a.pair ? a.H1 : 1);
    p.dh1 = make_div(a.H1);
    p.dk4 = make_div(a.Dm);
    p.da1 = make_div(a.Dq);
    if (a.q_outer) {
        p.din4 = make_div(a.G); p.aso = 1; p.asi = s.hm * s.rs; p.bso = (int)a.e2q; p.bsi = (int)a.e2g;
    } else {
        p.din4 = make_div(a.Dq); p.aso = s.hm * s.rs; p.asi = 1; p.bso = (int)a.e2g; p.bsi = (int)a.e2q;
    }
    const long long blocks = (long long)p.fblocks * a.batch;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_step64, dim3((unsigned)blocks), dim3(kStepNT), (size_t)s.lds, st, p);
    return hipGetLastError();
}

}  // namespace peps
