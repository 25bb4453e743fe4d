// Batched strided multi-index GEMM in float64 from registers.
//
// A float64 16x16x4 MFMA takes 64 cycles of its SIMD, so a wave that owns BM x BN blocks of
// 16 x 16 needs only BM + BN eight-byte loads per lane for 64 BM BN cycles of matrix work:
// operands go from memory (L1 and L2 hold the reuse) straight into MFMA operand registers,
// with no LDS tile, no barrier and no offset table, and waves run independently of each
// other.  Loads of the next KU k steps are in flight during the MFMAs of the current ones.
// Lane (li, gq) reads A(m0 + li, k0 + gq) and B(k0 + gq, n0 + li): 128-byte segments where
// the free index has unit stride, 32-byte ones (whose lines stay in L1 for the next steps)
// where k has it.  Multi-index offsets are 32-bit byte offsets from a wave-uniform base: one
// multiply-high per free index, an add and a carry per k step.
//
// Every output sums its products in ascending k in one MFMA chain (step s takes k = 4s ..
// 4s+3), as the LDS-staged kernel does: same bits for every tile shape and for both kernels.
//
// Bound by memory at short K, by the matrix cores at long K.  LDS-staged -> this kernel, us:
// two-row step at D = 6, bond 36, 64 samples, 1296 x 216 x 36 143 -> 47 (3.7 TB/s) and
// 7776 x 36 x 36 125 -> 70 (4.1 TB/s); 216 x 216 x 216, 256 samples 225 -> 149; D = 16, bond
// 32, 16 samples 16384 x 256 x 256 987 -> 645 (53 TFLOP/s); D = 4, bond 16, 4096 samples
// 1024 x 16 x 16 221 -> 178 (6 TB/s); the smallest products 4.6 -> 3.6 with their launch.
#include <algorithm>

#include "common.h"
#include "kernels.h"
#include "mfma_ops.h"

namespace peps {

namespace {

// offset of index i: i * si + (i / inner) * adj, in bytes, division by multiply-high
struct DMap {
    unsigned magic, si, adj;
};
// the same for k, walked in steps of 4: `step` bytes per step, `wrap` more when the inner
// index (advanced by `r4`) passes `inner`
struct DStep {
    DMap at;
    unsigned step, wrap;
    int inner, r4;
};
struct DgArgs {
    int M, N, K, batch, tiles_m, tiles_n;
    DMap am, bn, cm, cn;
    DStep ak, bk;
    long long a_bs, b_bs, c_bs;
    Gather ga, gb, gc;
    const double* A;
    const double* B;
    double* C;
    double alpha;
    int by_xcd;
    const int8_t* skip;
    long long skip_bs;
};

__device__ __forceinline__ unsigned dmap(const DMap& x, int i) {
    return (unsigned)i * x.si + __umulhi((unsigned)i, x.magic) * x.adj;
}
__device__ __forceinline__ double ld_byte(const double* p, unsigned off) {
    return *reinterpret_cast<const double*>(reinterpret_cast<const char*>(p) + off);
}

// running k offset of one operand
struct KWalk {
    unsigned off;
    int r;
};

template <int BM, int BN, int KU>
struct DFrag {
    double a[KU][BM], b[KU][BN];
};

template <int BM, int BN, int KU>
__device__ __forceinline__ void dg_load(DFrag<BM, BN, KU>& f, const DgArgs& g, const double* A, const double* B,
                                        const unsigned (&oa)[BM], const unsigned (&ob)[BN], KWalk& wa, KWalk& wb,
                                        int& k) {
#pragma unroll
    for (int u = 0; u < KU; ++u) {
        const bool in = k < g.K;
        const unsigned ka = in ? wa.off : 0, kb = in ? wb.off : 0;
#pragma unroll
        for (int i = 0; i < BM; ++i) f.a[u][i] = ld_byte(A, oa[i] + ka);
#pragma unroll
        for (int j = 0; j < BN; ++j) f.b[u][j] = ld_byte(B, ob[j] + kb);
        k += 4;
        wa.off += g.ak.step;
        wa.r += g.ak.r4;
        if (wa.r >= g.ak.inner) {
            wa.r -= g.ak.inner;
            wa.off += g.ak.wrap;
        }
        wb.off += g.bk.step;
        wb.r += g.bk.r4;
        if (wb.r >= g.bk.inner) {
            wb.r -= g.bk.inner;
            wb.off += g.bk.wrap;
        }
    }
}

// MFMAs of steps s0 .. s0 + KU - 1 (those below `steps`); past K (last step of a K that 4
// does not divide) both operands are zero
template <int BM, int BN, int KU>
__device__ __forceinline__ void dg_mul(mf64x4 (&acc)[BM][BN], DFrag<BM, BN, KU>& f, int s0, int steps, int K, int gq) {
#pragma unroll
    for (int u = 0; u < KU; ++u) {
        if (s0 + u >= steps) break;
        if (4 * (s0 + u) + 4 > K) {
            const bool in = 4 * (s0 + u) + gq < K;
#pragma unroll
            for (int i = 0; i < BM; ++i) f.a[u][i] = in ? f.a[u][i] : 0.0;
#pragma unroll
            for (int j = 0; j < BN; ++j) f.b[u][j] = in ? f.b[u][j] : 0.0;
        }
#pragma unroll
        for (int i = 0; i < BM; ++i)
#pragma unroll
            for (int j = 0; j < BN; ++j) acc[i][j] = mfma<Arith::F64>(f.a[u][i], f.b[u][j], acc[i][j]);
    }
}

template <int BM, int BN, int KU>
__global__ __launch_bounds__(256, (BM * BN >= 8 ? 2 : BM * BN >= 4 ? 3 : 4)) void k_dgemm(DgArgs g) {
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, gq = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    // workgroups go to the 8 XCDs in turn; g.by_xcd: each XCD takes one contiguous run of tiles, so
    // a sample's operands are fetched into one L2 only
    const unsigned nb = gridDim.x, per = nb / 8, rem = nb % 8, x = blockIdx.x % 8, y = blockIdx.x / 8;
    const unsigned blk = g.by_xcd ? x * per + (x < rem ? x : rem) + y : blockIdx.x;
    const unsigned t = blk * 4 + w, tiles = (unsigned)g.tiles_m * g.tiles_n;
    const int b = (int)(t / tiles);
    if (b >= g.batch) return;
    if (g.skip && g.skip[(long long)b * g.skip_bs] == 0) return;
    const int tt = (int)(t - (unsigned)b * tiles), tm = tt / g.tiles_n;
    const int m0 = tm * (16 * BM), n0 = (tt - tm * g.tiles_n) * (16 * BN);
    const double* A = g.A + (long long)b * g.a_bs + gather_off(g.ga, b);
    const double* B = g.B + (long long)b * g.b_bs + gather_off(g.gb, b);
    double* C = g.C + (long long)b * g.c_bs + gather_off(g.gc, b);

    unsigned oa[BM], ob[BN];   // rows and columns past the edge read the last valid one
#pragma unroll
    for (int i = 0; i < BM; ++i) oa[i] = dmap(g.am, min(m0 + 16 * i + li, g.M - 1));
#pragma unroll
    for (int j = 0; j < BN; ++j) ob[j] = dmap(g.bn, min(n0 + 16 * j + li, g.N - 1));
    int k = gq;
    const int qa = (int)__umulhi((unsigned)gq, g.ak.at.magic), qb = (int)__umulhi((unsigned)gq, g.bk.at.magic);
    KWalk wa{dmap(g.ak.at, gq), gq - qa * g.ak.inner}, wb{dmap(g.bk.at, gq), gq - qb * g.bk.inner};

    mf64x4 acc[BM][BN];
#pragma unroll
    for (int i = 0; i < BM; ++i)
#pragma unroll
        for (int j = 0; j < BN; ++j) acc[i][j] = mf64x4{0.0, 0.0, 0.0, 0.0};
    const int steps = (g.K + 3) / 4;
    DFrag<BM, BN, KU> f0, f1;
    dg_load<BM, BN, KU>(f0, g, A, B, oa, ob, wa, wb, k);
    for (int s = 0; s < steps; s += 2 * KU) {
        if (s + KU < steps) dg_load<BM, BN, KU>(f1, g, A, B, oa, ob, wa, wb, k);
        dg_mul<BM, BN, KU>(acc, f0, s, steps, g.K, gq);
        if (s + KU >= steps) break;
        if (s + 2 * KU < steps) dg_load<BM, BN, KU>(f0, g, A, B, oa, ob, wa, wb, k);
        dg_mul<BM, BN, KU>(acc, f1, s + KU, steps, g.K, gq);
    }

    unsigned oc[BN];
#pragma unroll
    for (int j = 0; j < BN; ++j) oc[j] = dmap(g.cn, n0 + 16 * j + li);
#pragma unroll
    for (int i = 0; i < BM; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = m0 + 16 * i + gq + 4 * r;
            const unsigned om = dmap(g.cm, m);
#pragma unroll
            for (int j = 0; j < BN; ++j) {
                if (m >= g.M || n0 + 16 * j + li >= g.N) continue;
                double* p = reinterpret_cast<double*>(reinterpret_cast<char*>(C) + (om + oc[j]));
                *p = g.alpha * acc[i][j][r];
            }
        }
}

// false when the division by multiply-high or the 32-bit byte offsets do not cover [0, n)
bool make_map(const Idx2& x, long long n, DMap& d, long long& bound) {
    if (x.inner <= 0 || x.s_outer < 0 || x.s_inner < 0) return false;
    long long inner = x.inner, si = x.s_inner;
    if (inner == 1) {
        inner = n;
        si = x.s_outer;
    }
    const bool split = inner < n;
    if (split && (n + 3) * inner >= (1LL << 32)) return false;
    bound += split ? (n - 1) / inner * x.s_outer + (inner - 1) * si : (n - 1) * si;
    d.magic = split ? (unsigned)((1LL << 32) / inner + 1) : 0u;
    d.si = (unsigned)(si * 8);
    d.adj = split ? (unsigned)((x.s_outer - inner * si) * 8) : 0u;
    return true;
}
bool make_step(const Idx2& x, int n, DStep& d, long long& bound) {
    if (!make_map(x, n, d.at, bound)) return false;
    long long inner = x.inner, si = x.s_inner;
    if (inner == 1) {
        inner = n;
        si = x.s_outer;
    }
    if (inner >= n) {   // one index: no carry
        d.inner = 1 << 30;
        d.r4 = 0;
        d.step = (unsigned)(4 * si * 8);
        d.wrap = 0;
        return true;
    }
    d.inner = (int)inner;
    d.r4 = (int)(4 % inner);
    d.step = (unsigned)((4 / inner * x.s_outer + 4 % inner * si) * 8);
    d.wrap = (unsigned)((x.s_outer - inner * si) * 8);
    return true;
}

// An operand whose 16 x 4 loads fall on 64 separate lines: neither the free index nor k has unit
// stride, and a line comes back only after the `inner` values of k (the site products of a backward
// step).  With 6 of them the lines stay in L1 and this kernel is the faster (36 x 7776 x 36, 64 samples
// 78 us, LDS-staged 120), with 8 it is not (64 x 32768 x 64, 32 samples 357 and 345), with 16 far from
// it (256 x 16384 x 256, 16 samples 4.8 and 2.2 ms).  Read for at most 64 rows of the other operand
// the lines hardly come back anyway, and the more numerous waves win (32 x 512 x 512, 16 samples
// 24 and 64 us).
bool scattered(const Idx2& free, int n, const Idx2& k, int nk, int other) {
    const auto inner = [](const Idx2& x, int m) { return x.inner == 1 ? m : std::min(x.inner, m); };
    const auto stride = [](const Idx2& x) { return x.inner == 1 ? x.s_outer : x.s_inner; };
    return other > 64 && inner(free, n) >= 8 && stride(free) > 1 && inner(k, nk) >= 8 && stride(k) > 1;
}

}  // namespace

bool gemm_scattered(const GemmArgs& g) {
    return scattered(g.am, g.M, g.ak, g.K, g.N) || scattered(g.bn, g.N, g.bk, g.K, g.M);
}

namespace {

// Samples a multiple of 32 KB apart: runs of tiles by XCD would start on the same memory channel
// (D = 16, bond 32, 16 samples: a product of 328 us takes 1226).  Elsewhere runs by XCD gain up to a
// fifth (216 x 216 x 36, 256 samples 33 us, 40 in turn).
bool camps(long long bs) { return bs != 0 && bs % 4096 == 0; }

bool make_args(const GemmArgs& g, DgArgs& d) {
    if (g.a_f32 || g.b_f32 || g.c_f32 || g.beta != 0.0 || g.K <= 0) return false;
    if (gemm_scattered(g)) return false;
    long long ba = 0, bb = 0, bc = 0;
    // rows are mapped up to the end of their tile on the output side (masked there)
    if (!make_map(g.am, g.M, d.am, ba) || !make_map(g.bn, g.N, d.bn, bb) || !make_map(g.cm, g.M, d.cm, bc) ||
        !make_map(g.cn, g.N, d.cn, bc) || !make_step(g.ak, g.K, d.ak, ba) || !make_step(g.bk, g.K, d.bk, bb))
        return false;
    if (std::max(ba, std::max(bb, bc)) >= (1LL << 29)) return false;
    d.M = g.M; d.N = g.N; d.K = g.K; d.batch = g.batch;
    d.a_bs = g.a_bs; d.b_bs = g.b_bs; d.c_bs = g.c_bs;
    d.ga = g.ga; d.gb = g.gb; d.gc = g.gc;
    d.A = g.A; d.B = g.B; d.C = g.C;
    d.alpha = g.alpha;
    d.by_xcd = !(camps(g.a_bs) || camps(g.b_bs) || camps(g.c_bs));
    d.skip = g.skip; d.skip_bs = g.skip_bs;
    return true;
}

template <int BM, int BN>
hipError_t launch_d(DgArgs& d, hipStream_t st) {
    d.tiles_m = (d.M + 16 * BM - 1) / (16 * BM);
    d.tiles_n = (d.N + 16 * BN - 1) / (16 * BN);
    const long long waves = (long long)d.tiles_m * d.tiles_n * d.batch, blocks = (waves + 3) / 4;
    if (blocks > 0x3fffffffLL) return hipErrorInvalidValue;
    const int steps = (d.K + 3) / 4;
    if (steps % 3 == 0 && steps % 4 != 0)
        hipLaunchKernelGGL((k_dgemm<BM, BN, 3>), dim3((unsigned)blocks), dim3(256), 0, st, d);
    else
        hipLaunchKernelGGL((k_dgemm<BM, BN, 4>), dim3((unsigned)blocks), dim3(256), 0, st, d);
    return hipGetLastError();
}

// Cost (cycles) of a launch with BM x BN blocks per wave: a wave's MFMAs (64 each), loads and
// stores, times the waves of the fullest of the 1024 SIMDs (counted in halves), plus the
// load latency of the first.  Fitted to 12 shapes of blocks over 168 products (D = 2 to 16,
// bonds 4 to 64, 1 to 8192 samples): on average within 2 % of the fastest shape of blocks.
long long wave_cost(const DgArgs& d, int bm, int bn) {
    const long long waves = (long long)((d.M + 16 * bm - 1) / (16 * bm)) * ((d.N + 16 * bn - 1) / (16 * bn)) * d.batch;
    const long long steps = (d.K + 3) / 4, halves = std::max(2LL, (waves + 511) / 512);
    return 2 * (steps * (64 * bm * bn + 37) + 50 * bm * bn) +
           (halves - 2) * (steps * (64 * bm * bn + 11 * (bm + bn)) + 50 * bm * bn);
}

}  // namespace

hipError_t launch_dgemm(const GemmArgs& g, hipStream_t st, bool& done) {
    DgArgs d;
    done = make_args(g, d);
    if (!done) return hipSuccess;
    constexpr int shapes[12][2] = {{1, 1}, {2, 1}, {1, 2}, {2, 2}, {1, 3}, {3, 1},
                                   {2, 3}, {3, 2}, {2, 4}, {4, 2}, {3, 4}, {4, 3}};
    int best = 0;
    for (int i = 1; i < 12; ++i)
        if (wave_cost(d, shapes[i][0], shapes[i][1]) < wave_cost(d, shapes[best][0], shapes[best][1])) best = i;
    switch (best) {
        case 0: return launch_d<1, 1>(d, st);
        case 1: return launch_d<2, 1>(d, st);
        case 2: return launch_d<1, 2>(d, st);
        case 3: return launch_d<2, 2>(d, st);
        case 4: return launch_d<1, 3>(d, st);
        case 5: return launch_d<3, 1>(d, st);
        case 6: return launch_d<2, 3>(d, st);
        case 7: return launch_d<3, 2>(d, st);
        case 8: return launch_d<2, 4>(d, st);
        case 9: return launch_d<4, 2>(d, st);
        case 10: return launch_d<3, 4>(d, st);
        default: return launch_d<4, 3>(d, st);
    }
}

}  // namespace peps
