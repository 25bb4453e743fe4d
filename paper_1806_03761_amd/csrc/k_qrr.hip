// Triangular factors of tall column tensors in float64: R of X = Q R for the left-to-right
// sweep of the truncation (Fig. 1(c)), where the right-to-left sweep needs no Q (k_trunc.hip).
//
// X is row-major m x n.  Blocked Householder, right-looking, in panels of 32 columns (16 where
// more than 1408 rows are left):
//   k_qrr_panel   one workgroup per matrix: the panel in registers, in the accumulator layout
//                 of the 16x16x4 MFMA (lane (li, gq): column li, rows gq + 4 r of a tile), so a
//                 dot product over the rows is a sum inside the lane, two lane exchanges
//                 and one LDS pass over the eight waves, and U^T U reads the registers as MFMA
//                 operands; one barrier per column;
//   k_qrr_update  one workgroup per (matrix, block of as many trailing columns): the block in
//                 registers in the same layout, W = U^T A, A -= U (T^T W) on the matrix cores;
//                 the block is read and written once, its first rows leave as rows of R.
// The reflectors are left unnormalised, H = I - t u u^T with u = (alpha - beta, x): no column is
// rescaled, T carries the factors.  R is not rescaled either: by its leading entry, a first column
// far below the others would carry them out of range.
// Taller matrices are cut into blocks of up to 2048 rows, factorised side by side, and their
// R factors, stacked, factorised again.
//
// Bound: the panel by its chain of columns (about 0.5 us of exchange and scalars each, and 0.1 us
// per 128 rows), the update by memory (3 TB/s).  1296 x 216: 256 matrices 3.6 ms with 16-column
// panels, T matrices merged in pairs and three GEMMs per pair, 2.0 ms so; 48 matrices 2.0 and
// 0.92 ms.
#include <algorithm>

#include "common.h"
#include "kernels.h"
#include "householder.h"

namespace peps {

namespace {

typedef double d4v __attribute__((ext_vector_type(4)));

constexpr int kQrrNW = 8;            // waves of both kernels
constexpr int kQrrRows2 = 1408;      // tallest panel of 32 columns (11 tiles of 16 rows per wave)
constexpr int kQrrRows1 = 2048;      // tallest panel of 16 columns
constexpr int kQrrT = 32 * 32 + 16;  // doubles of a T in the scratch

struct QrrArgs {
    double* X; long long xs;         // matrix b: sub-block h = b % nsub of X + (b / nsub) xs
    int m, n, nsub, mb;              // rows and columns; rows of a sub-block
    int rblk; long long rstr;        // row i lies at (i / rblk) rstr + i % rblk (rblk = 0: at i)
    double* R; long long rs, rsub;   // R of matrix b at R + (b / nsub) rs + (b % nsub) rsub, ld n
    double* V; long long vs, vsub;   // packed reflectors of the current panel, and behind them
    long long ot;                    // (at ot) its T, 32 x 32 row-major
    int nmat;
};

__device__ __forceinline__ double* qrr_v(const QrrArgs& q, int b) {
    return q.V + (long long)(b / q.nsub) * q.vs + (long long)(b % q.nsub) * q.vsub;
}

__device__ __forceinline__ void qrr_matrix(const QrrArgs& q, int b, double*& X, double*& R, int& m) {
    const int h = b % q.nsub;
    X = q.X + (long long)(b / q.nsub) * q.xs + (long long)h * q.mb * q.n;
    R = q.R + (long long)(b / q.nsub) * q.rs + (long long)h * q.rsub;
    m = min(q.mb, q.m - h * q.mb);
}

template <bool MAP>
__device__ __forceinline__ long long qrr_row(const QrrArgs& q, int i) {
    if constexpr (MAP) return ((long long)(i / q.rblk) * q.rstr + i % q.rblk) * q.n;
    else return (long long)i * q.n;
}

// The value of lane L of every row of 16 lanes, in all of them (two 32-bit DPP moves: the 64-bit
// one runs at a quarter of their rate).
template <int L>
__device__ __forceinline__ double row_bcast(double x) {
    const long long v = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_mov_dpp((int)v, 0x150 + L, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(v >> 32), 0x150 + L, 0xF, 0xF, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// The factorisation of one 16-column tile x.  The column index is a template argument, since the
// broadcast of the pivot column across a row of lanes is a DPP move with a constant lane.
template <int RT>
struct QrrTile {
    static constexpr int NW = kQrrNW;
    double x[RT][4];
    double (*red)[NW][16];
    double (*prow)[16];
    double *rd, *tp;   // of this tile
    int w, li, gq, row0, nref;   // row0: the tile's first pivot row inside the panel (a multiple of 16)

    // Steps LJ .. 15; returns the first column left out, one whose squares do not fit the range of doubles.
    template <int LJ>
    __device__ __forceinline__ int step() {
        if constexpr (LJ < 16) {
            constexpr int par = LJ & 1, le = LJ >> 2;
            if (LJ >= nref) return 16;   // uniform
            const bool owner = 16 * w == row0 && gq == (LJ & 3);   // lanes holding the pivot row
            if (owner) prow[par][li] = x[0][le];
            double y0[4];   // the pivot column of the first row tile, zero down to the pivot
#pragma unroll
            for (int e = 0; e < 4; ++e) y0[e] = 16 * w + gq + 4 * e > row0 + LJ ? x[0][e] : 0.0;
            double s[2] = {0.0, 0.0};
#pragma unroll
            for (int t = 0; t < RT; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    s[e & 1] = fma(row_bcast<LJ>(t == 0 ? y0[e] : x[t][e]), x[t][e], s[e & 1]);
            const double d = add_xor32(add_xor16(s[0] + s[1]));
            if (gq == 0) red[par][w][li] = d;
            __syncthreads();
            const auto total = [&](int col) -> double {
                const double(*p)[16] = red[par];
                return ((p[0][col] + p[1][col]) + (p[2][col] + p[3][col])) +
                       ((p[4][col] + p[5][col]) + (p[6][col] + p[7][col]));
            };
            const double sq = total(LJ), al = prow[par][LJ], ta = total(li), pa = prow[par][li];
            double be, up, tq;
            if (!hh_unnormalised(al, sq, be, up, tq)) return LJ;
            const double f = li > LJ ? tq * fma(up, pa, ta) : 0.0;
            if (threadIdx.x == 0) {
                rd[LJ] = be;
                tp[LJ] = tq;
            }
            // lane LJ, the source of the broadcasts, has f = 0 and keeps its column
#pragma unroll
            for (int t = 0; t < RT; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    // broadcast again: the values of the tallest tiles would not fit beside them
                    if (RT > 11 && t > 0) asm volatile("" : "+v"(x[t][e]));
                    x[t][e] = fma(-f, row_bcast<LJ>(t == 0 ? y0[e] : x[t][e]), x[t][e]);
                }
            if (owner) x[0][le] = li == LJ ? up : fma(-f, up, x[0][le]);
            return step<LJ + 1>();
        }
        return 16;
    }

    // The columns j0 .. nref - 1 at any scale: u is brought to order one by a power of two.  One rolled
    // loop, with the column in LDS: handled inside the unrolled steps it cost 1 % of a 16x16 D = 6
    // amplitude, in code alone.
    __device__ __forceinline__ void steps_scaled(int j0, double* col) {
        col += 16 * w + gq;   // entry (t, e) of this lane's column at 16 NW t + 4 e
#pragma clang loop unroll(disable)
        for (int j = j0; j < nref; ++j) {
            const int le = j >> 2, pivot = row0 + j - 16 * w - gq;   // entry e of tile 0 is below it for 4 e > pivot
            const bool owner = 16 * w == row0 && gq == (j & 3);
            double mx = 0.0;   // the largest entry of the column
            if (li == j) {
#pragma unroll
                for (int t = 0; t < RT; ++t)
#pragma unroll
                    for (int e = 0; e < 4; ++e) mx = t > 0 || 4 * e >= pivot ? fmax(mx, fabs(x[t][e])) : mx;
            }
            for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o, 64));
            __syncthreads();
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (owner && e == le) prow[0][li] = x[0][e];
            if (li == 0 && gq == 0) red[0][w][0] = mx;
            __syncthreads();
            for (int v = 0; v < NW; ++v) mx = fmax(mx, red[0][v][0]);
            const int ex = mx > 0.0 && mx < INFINITY ? -__builtin_amdgcn_frexp_exp(mx) : 0;
            if (li == j) {
#pragma unroll
                for (int t = 0; t < RT; ++t)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const bool below = t > 0 || 4 * e > pivot;
                        x[t][e] = __builtin_amdgcn_ldexp(x[t][e], below ? ex : 0);
                        col[16 * NW * t + 4 * e] = below ? x[t][e] : 0.0;
                    }
            }
            __syncthreads();
            double s = 0.0;
#pragma unroll
            for (int t = 0; t < RT; ++t) {
#pragma unroll
                for (int e = 0; e < 4; ++e) s = fma(col[16 * NW * t + 4 * e], x[t][e], s);
                asm volatile("" : "+v"(s)::"memory");   // one tile's reads at a time
            }
            s = add_xor32(add_xor16(s));
            if (gq == 0) red[1][w][li] = s;
            __syncthreads();
            double sq = 0.0, ta = 0.0;
            for (int v = 0; v < NW; ++v) {
                sq += red[1][v][j];
                ta += red[1][v][li];
            }
            const double al = __builtin_amdgcn_ldexp(prow[0][j], ex);
            const double nrm = sqrt(fma(al, al, sq)), up = sq == 0.0 ? 0.0 : al + copysign(nrm, al);
            const double tq = sq == 0.0 ? 0.0 : 1.0 / (nrm * (nrm + fabs(al)));
            const double f = li > j ? tq * fma(up, prow[0][li], ta) : 0.0;
            if (threadIdx.x == 0) {
                rd[j] = sq == 0.0 ? prow[0][j] : __builtin_amdgcn_ldexp(-copysign(nrm, al), -ex);
                tp[j] = tq;
            }
#pragma unroll
            for (int t = 0; t < RT; ++t) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    x[t][e] = fma(-f, col[16 * NW * t + 4 * e], x[t][e]);
                    if (t == 0 && owner && e == le) x[0][e] = li == j ? up : fma(-f, up, x[0][e]);
                }
                asm volatile("" ::: "memory");
            }
        }
    }
};

template <int RT, int CT, bool MAP>
__global__ __launch_bounds__(64 * kQrrNW) void k_qrr_panel(QrrArgs q, int k0) {
    constexpr int NW = kQrrNW, PW = 16 * CT, CH = RT < 6 ? RT : 6;   // CH row tiles' reflectors in flight
    __shared__ double red[2][NW][16], prow[2][16], rd[16], tp[16];
    __shared__ double part[NW * 256], Gs[CT][256], Tl[CT][256], Wl[256];
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = tid >> 6, li = lane & 15, gq = lane >> 4;
    double *X, *R;
    int m;
    qrr_matrix(q, b, X, R, m);
    const int n = q.n, r = min(m, n);
    if (k0 >= r) return;
    const int nc = min(PW, n - k0), nref = min(PW, r - k0);
    double* Vb = qrr_v(q, b);
    double* Tb = Vb + q.ot;
    const int nt = (m - k0 + 15) / 16;   // row tiles
    // first reflector tile of this wave's row tile t (the last one's past the end)
    const auto tile = [&](int t) { return Vb + (long long)min(w + NW * t, nt - 1) * CT * 256; };
    double* Rk = R + (long long)k0 * n;
    QrrTile<RT> p;
    p.red = red; p.prow = prow; p.rd = rd; p.tp = tp;
    p.w = w; p.li = li; p.gq = gq;
    auto& x = p.x;
    // sum of the waves' 16 x 16 partial products in `part`, element tid (tid < 256) to dst
    const auto gather = [&](double* dst) {
        __syncthreads();
        if (tid < 256) {
            double s = 0.0;
#pragma unroll
            for (int v = 0; v < NW; ++v) s += part[v * 256 + tid];
            dst[tid] = s;
        }
        __syncthreads();
    };
    const auto scatter = [&](const d4v& acc) {
#pragma unroll
        for (int e = 0; e < 4; ++e) part[w * 256 + (gq + 4 * e) * 16 + li] = acc[e];
    };
    // the tiles in turn, through the same code: the first one's reflectors reach the second as a
    // WY update on the matrix cores, and only one tile is held in registers
    const auto load_tile = [&](int c) {
        const int col = 16 * c + li;
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int i = k0 + 16 * (w + NW * t) + gq + 4 * e;
                x[t][e] = ld_or0(i < m && col < nc, X, qrr_row<MAP>(q, i < m ? i : 0) + k0 + col);
            }
    };
    load_tile(0);
#pragma clang loop unroll(disable)
    for (int c = 0; c < CT; ++c) {
        const int tref = max(0, min(16, nref - 16 * c)), col = 16 * c + li;
        p.row0 = 16 * c;
        p.nref = tref;
        if (CT == 2 && c == 1) {
            // x -= U0 T0^T (U0^T x)
            d4v acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int t0 = 0; t0 < RT; t0 += CH) {
                double v[CH][4];
#pragma unroll
                for (int t = t0; t < t0 + CH && t < RT; ++t)
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[t - t0][e] = tile(t)[(gq + 4 * e) * 16 + li];
#pragma unroll
                for (int t = t0; t < t0 + CH && t < RT; ++t)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(v[t - t0][e], x[t][e], acc, 0, 0, 0);
            }
            scatter(acc);
            gather(Wl);
            double v2 = 0.0;
            if (tid < 256) {
#pragma unroll
                for (int k = 0; k < 16; ++k) v2 = fma(Tl[0][k * 16 + (tid >> 4)], Wl[k * 16 + (tid & 15)], v2);
            }
            __syncthreads();
            if (tid < 256) Wl[tid] = v2;
            __syncthreads();
#pragma unroll
            for (int t0 = 0; t0 < RT; t0 += CH) {
                double v[CH][4];
#pragma unroll
                for (int t = t0; t < t0 + CH && t < RT; ++t)
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[t - t0][e] = -tile(t)[li * 16 + 4 * gq + e];
#pragma unroll
                for (int t = t0; t < t0 + CH && t < RT; ++t) {
                    d4v a = {x[t][0], x[t][1], x[t][2], x[t][3]};
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        a = __builtin_amdgcn_mfma_f64_16x16x4f64(v[t - t0][e], Wl[(4 * gq + e) * 16 + li], a, 0, 0, 0);
                    const bool live = w + NW * t < nt;   // rows past the last tile stay zero
#pragma unroll
                    for (int e = 0; e < 4; ++e) x[t][e] = live ? a[e] : 0.0;
                }
            }
        }
        if (const int j = p.template step<0>(); j < 16) p.steps_scaled(j, part);   // uniform
        __syncthreads();
        // the tile's part of the rows k0 .. of R, then zeros above the pivots of U
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = 16 * w + gq + 4 * e;   // inside the panel (t = 0)
            if (i < nref && col < nc) Rk[(long long)i * n + k0 + col] = col > i ? x[0][e] : (col == i ? rd[li] : 0.0);
            if (i < col) x[0][e] = 0.0;
        }
        if (li >= tref) {
#pragma unroll
            for (int t = 0; t < RT; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e) x[t][e] = 0.0;
        }
        if (k0 + nc >= n && c == CT - 1) break;   // no column left that needs this tile's reflectors
        // U packed: tile (row tile, column tile) row-major 16 x 16; U^T U, and U0^T U1
        d4v acc = {0.0, 0.0, 0.0, 0.0}, acc01 = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            if (w + NW * t < nt) {
                double* vp = Vb + ((long long)(w + NW * t) * CT + c) * 256;
#pragma unroll
                for (int e = 0; e < 4; ++e) vp[(gq + 4 * e) * 16 + li] = x[t][e];
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(x[t][e], x[t][e], acc, 0, 0, 0);
        }
        if (CT == 2 && c == 1) {
#pragma unroll
            for (int t0 = 0; t0 < RT; t0 += CH) {
                double v[CH][4];
#pragma unroll
                for (int t = t0; t < t0 + CH && t < RT; ++t)
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[t - t0][e] = tile(t)[(gq + 4 * e) * 16 + li];
#pragma unroll
                for (int t = t0; t < t0 + CH && t < RT; ++t)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        acc01 = __builtin_amdgcn_mfma_f64_16x16x4f64(v[t - t0][e], x[t][e], acc01, 0, 0, 0);
            }
        }
        scatter(acc);
        if (CT == 2 && c == 0) load_tile(1);   // in flight while T is formed
        gather(Gs[0]);
        if (CT == 2 && c == 1) {
            scatter(acc01);
            gather(Gs[CT - 1]);
        }
        // T of the tile: T_jj = t_j, T[0:j, j] = -t_j T[0:j, 0:j] (U^T U)[0:j, j]; row i needs only its
        // own earlier entries
        if (tid < 16) {
            double row[16], g[16], gn[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) g[j] = row[j] = 0.0;
#pragma unroll
            for (int j = 0; j < 16; ++j) {
#pragma unroll
                for (int k = 0; k < 16; ++k)
                    if (k <= j && j + 1 < 16) gn[k] = Gs[0][k * 16 + j + 1];   // the next column's reads in flight
                double s0 = 0.0, s1 = 0.0;
#pragma unroll
                for (int k = 0; k < 16; k += 2) {
                    if (k < j) s0 = fma(row[k], g[k], s0);   // row[k] = 0 for k < tid
                    if (k + 1 < j) s1 = fma(row[k + 1], g[k + 1], s1);
                }
                const double tj = j < tref ? tp[j] : 0.0;
                row[j] = j < tid ? 0.0 : (j == tid ? tj : -tj * (s0 + s1));
                asm volatile("" : "+v"(row[j])::"memory");   // no more than one column ahead
#pragma unroll
                for (int k = 0; k < 16; ++k)
                    if (k <= j) g[k] = gn[k];
            }
#pragma unroll
            for (int j = 0; j < 16; ++j) Tl[c][tid * 16 + j] = row[j];
        }
        __syncthreads();
    }
    for (int e = tid; e < nref * k0; e += 64 * NW) Rk[(long long)(e / k0) * n + e % k0] = 0.0;   // left of the panel
    if (CT == 2 && nref > 16)   // rows of the second tile, columns of the first
        for (int e = tid; e < (nref - 16) * 16; e += 64 * NW) Rk[(long long)(16 + e / 16) * n + k0 + e % 16] = 0.0;
    if (k0 + nc >= n) return;   // no trailing column
    const int a = (tid >> 4) & 15, c = tid & 15;
    if constexpr (CT == 1) {
        if (tid < 256) Tb[a * 32 + c] = Tl[0][tid];
    } else {   // [[T1, -T1 (U0^T U1) T2], [0, T2]]
        if (tid < 256) {
            double s = 0.0;
#pragma unroll
            for (int k = 0; k < 16; ++k) s = fma(Gs[1][a * 16 + k], Tl[1][k * 16 + c], s);
            Wl[tid] = s;
        }
        __syncthreads();
        if (tid < 256) {
            double s = 0.0;
#pragma unroll
            for (int k = 0; k < 16; ++k) s = fma(Tl[0][a * 16 + k], Wl[k * 16 + c], s);
            Tb[a * 32 + c] = Tl[0][tid];
            Tb[a * 32 + 16 + c] = -s;
            Tb[(16 + a) * 32 + c] = 0.0;
            Tb[(16 + a) * 32 + 16 + c] = Tl[1][tid];
        }
    }
}

// Blocks of one matrix are given to one XCD (workgroups go round the 8 XCDs), whose L2 then
// holds its reflectors for all of them.  One workgroup per CU, since the block fills the
// registers; smaller blocks or a second read of it, with two workgroups per CU, were slower
// (1296 rows, 256 matrices, 184 trailing columns: 358 us so, 716 us with 16-column blocks, 492 us
// streaming the block twice with one row tile ahead).
template <int RT, int CT, bool MAP>
__global__ __launch_bounds__(64 * kQrrNW) void k_qrr_update(QrrArgs q, int k0, int cblocks) {
    constexpr int NW = kQrrNW, PW = 16 * CT, LW = PW + 1;
    extern __shared__ __align__(16) double sh[];   // NW x CT x CT x 256 partial sums
    __shared__ double Ws[PW * LW], W2[PW * LW];
    const int loc = blockIdx.x / 8, b = (loc / cblocks) * 8 + blockIdx.x % 8, cb = loc % cblocks;
    if (b >= q.nmat) return;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, li = lane & 15, gq = lane >> 4;
    double *X, *R;
    int m;
    qrr_matrix(q, b, X, R, m);
    const int n = q.n, r = min(m, n), c0 = k0 + PW + PW * cb;
    if (k0 >= r || c0 >= n) return;
    const double* Vb = qrr_v(q, b) + (long long)w * CT * 256;
    const double* Tb = qrr_v(q, b) + q.ot;
    const int nt = (m - k0 + 15) / 16;
    double x[RT][CT][4];
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = k0 + 16 * (w + NW * t) + gq + 4 * e;
            const long long ro = qrr_row<MAP>(q, i < m ? i : 0) + c0;
#pragma unroll
            for (int c = 0; c < CT; ++c) x[t][c][e] = ld_or0(i < m && c0 + 16 * c + li < n, X, ro + 16 * c + li);
        }
    d4v wp[CT][CT];
#pragma unroll
    for (int a = 0; a < CT; ++a)
#pragma unroll
        for (int c = 0; c < CT; ++c) wp[a][c] = d4v{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        if (w + NW * t >= nt) continue;   // uniform over the wave
        double v[CT][4];
#pragma unroll
        for (int a = 0; a < CT; ++a)
#pragma unroll
            for (int e = 0; e < 4; ++e) v[a][e] = Vb[(NW * t * CT + a) * 256 + (gq + 4 * e) * 16 + li];
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int a = 0; a < CT; ++a)
#pragma unroll
                for (int c = 0; c < CT; ++c)
                    wp[a][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(v[a][e], x[t][c][e], wp[a][c], 0, 0, 0);
    }
#pragma unroll
    for (int a = 0; a < CT; ++a)
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                sh[((w * CT + a) * CT + c) * 256 + (gq + 4 * e) * 16 + li] = wp[a][c][e];
    __syncthreads();
    for (int e = tid; e < CT * CT * 256; e += 64 * NW) {
        double s = 0.0;
#pragma unroll
        for (int v = 0; v < NW; ++v) s += sh[v * CT * CT * 256 + e];
        const int a = e / (CT * 256), c = (e / 256) % CT, i = (e >> 4) & 15, k = e & 15;
        Ws[(16 * a + i) * LW + 16 * c + k] = s;
    }
    __syncthreads();
    if (w < CT * CT) {   // W2 = T^T W, one tile per wave
        const int a = w / CT, c = w % CT;
        d4v acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int s = 0; s < 4 * CT; ++s) {
            const int k = 4 * s + gq;
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(Tb[k * 32 + 16 * a + li], Ws[k * LW + 16 * c + li], acc, 0, 0, 0);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) W2[(16 * a + gq + 4 * e) * LW + 16 * c + li] = acc[e];
    }
    __syncthreads();
    // step s takes the reflectors 4 gq + s: a lane reads four consecutive ones of its row
    const auto load_u = [&](int t, double (&v)[CT][4]) {
        const int tt = w + NW * t < nt ? NW * t : 0;
#pragma unroll
        for (int a = 0; a < CT; ++a)
#pragma unroll
            for (int s = 0; s < 4; ++s) v[a][s] = Vb[(tt * CT + a) * 256 + li * 16 + 4 * gq + s];
    };
    double v[CT][4];
    load_u(0, v);
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        double vn[CT][4];   // the next row tile's, in flight
        if (t + 1 < RT) load_u(t + 1, vn);
        if (w + NW * t < nt) {
            d4v acc[CT];
#pragma unroll
            for (int c = 0; c < CT; ++c) acc[c] = d4v{x[t][c][0], x[t][c][1], x[t][c][2], x[t][c][3]};
#pragma unroll
            for (int a = 0; a < CT; ++a)
#pragma unroll
                for (int s = 0; s < 4; ++s)
#pragma unroll
                    for (int c = 0; c < CT; ++c)
                        acc[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(
                            -v[a][s], W2[(16 * a + 4 * gq + s) * LW + 16 * c + li], acc[c], 0, 0, 0);
            // the panel's own rows are rows of R, the others go on
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int i = 16 * (w + NW * t) + gq + 4 * e;
                if (k0 + i >= m) continue;
                const bool fin = t == 0 && i < min(PW, r - k0);
                double* row = fin ? R + (long long)(k0 + i) * n : X + qrr_row<MAP>(q, k0 + i);
#pragma unroll
                for (int c = 0; c < CT; ++c)
                    if (c0 + 16 * c + li < n)
                        row[c0 + 16 * c + li] = acc[c][e];
            }
        }
        if (t + 1 < RT) {
#pragma unroll
            for (int a = 0; a < CT; ++a)
#pragma unroll
                for (int s = 0; s < 4; ++s) v[a][s] = vn[a][s];
        }
    }
}

template <int RT, int CT, bool MAP>
hipError_t qrr_step(const QrrArgs& q, int k0, hipStream_t st) {
    constexpr int PW = 16 * CT;
    hipLaunchKernelGGL((k_qrr_panel<RT, CT, MAP>), dim3(q.nmat), dim3(64 * kQrrNW), 0, st, q, k0);
    const int trail = q.n - (k0 + PW);
    if (trail > 0) {
        const int cblocks = (trail + PW - 1) / PW;
        hipLaunchKernelGGL((k_qrr_update<RT, CT, MAP>), dim3((unsigned)((q.nmat + 7) / 8 * 8 * cblocks)),
                           dim3(64 * kQrrNW), (size_t)kQrrNW * CT * CT * 256 * sizeof(double), st, q, k0, cblocks);
    }
    return hipGetLastError();
}

// The height of a panel is the number of 16-row tiles per wave (128 rows each), a launch of its own.  A
// panel of 1024 matrices takes 104 us with one, 152 with two, 399 with nine and 538 with eleven, so a
// spare tile costs 8 to 13 % of it.  Above 1024 rows, where a tall tensor spends most of its panels,
// every height is there; below, where a panel is cheap and only few are left, every second one.
template <bool MAP>
hipError_t qrr_run(const QrrArgs& q, hipStream_t st) {
    const int rows = q.nsub > 1 ? q.mb : q.m, r = std::min(rows, q.n);
    for (int k0 = 0; k0 < r;) {
        const int left = rows - k0;
        hipError_t e;
        if (left > kQrrRows2) {
            e = qrr_step<16, 1, MAP>(q, k0, st);
            k0 += 16;
        } else {
            if (left <= 128) e = qrr_step<1, 2, MAP>(q, k0, st);
            else if (left <= 256) e = qrr_step<2, 2, MAP>(q, k0, st);
            else if (left <= 512) e = qrr_step<4, 2, MAP>(q, k0, st);
            else if (left <= 768) e = qrr_step<6, 2, MAP>(q, k0, st);
            else if (left <= 1024) e = qrr_step<8, 2, MAP>(q, k0, st);
            else if (left <= 1152) e = qrr_step<9, 2, MAP>(q, k0, st);
            else if (left <= 1280) e = qrr_step<10, 2, MAP>(q, k0, st);
            else e = qrr_step<11, 2, MAP>(q, k0, st);
            k0 += 32;
        }
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

int qrr_blocks(int m) { return m <= kQrrRows1 ? 1 : (m + kQrrRows1 - 1) / kQrrRows1; }

}  // namespace

// One packed panel and one T per row block, and 16 doubles: panels a multiple of 4 KB apart would all
// start on the same memory channels (update of 1296-row matrices, 256 of them: 188 us, 192 without).
long long qrr_scratch_doubles(int m) {
    const int s = qrr_blocks(m), mb = std::min(m, kQrrRows1);
    return s * ((long long)((mb + 15) / 16) * 512 + kQrrT);
}

bool qrr_fits(int m, int n) {
    const int s = qrr_blocks(m);
    if (m < 1 || n < 1) return false;
    if (s == 1) return true;
    const int mb = ((m + s - 1) / s + 15) / 16 * 16;
    return m - (s - 1) * mb >= n && s * n <= kQrrRows1;   // every block has its n rows of R, stacked once
}

hipError_t launch_qr_r(double* X, long long xs, int m, int n, double* R, long long rs, double* W, long long ws,
                       int batch, hipStream_t st) {
    if (batch <= 0) return hipSuccess;
    if (!qrr_fits(m, n) || ws < qrr_scratch_doubles(m)) return hipErrorInvalidValue;
    const int s = qrr_blocks(m);
    QrrArgs q{};
    q.X = X; q.xs = xs; q.n = n; q.m = m;
    q.V = W; q.vs = ws;
    q.ot = (long long)((std::min(m, kQrrRows1) + 15) / 16) * 512;
    q.vsub = q.ot + kQrrT;
    if (s == 1) {
        q.mb = m;
        q.nsub = 1;
        q.R = R; q.rs = rs;
        q.nmat = batch;
        return qrr_run<false>(q, st);
    }
    // the blocks side by side, each R over its block's first n rows; then those stacked
    q.mb = ((m + s - 1) / s + 15) / 16 * 16;
    q.nsub = s;
    q.R = X; q.rs = xs; q.rsub = (long long)q.mb * n;
    q.nmat = batch * s;
    hipError_t e = qrr_run<false>(q, st);
    if (e != hipSuccess) return e;
    QrrArgs p = q;
    p.m = p.mb = s * n;
    p.rblk = n; p.rstr = q.mb;
    p.nsub = 1;
    p.R = R; p.rs = rs; p.rsub = 0;
    p.nmat = batch;
    return qrr_run<true>(p, st);
}

}  // namespace peps
