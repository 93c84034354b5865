// Batched blocked Gauss-Jordan inversion with partial pivoting (setup of the factorised K^{-1}
// and of the complete-inverse correction).
//
// The matrix is inverted in place in panels of GJ_NB columns.  A panel's columns c are
// eliminated for all rows; the other columns then receive the elimination at once, as two
// products with the panel's rows r and columns c:
//     A[not r, not c] += A[not r, c] A[r, not c]        (old A[r, not c])
//     A[r, not c]      = A[r, c] A[r, not c]
// The row swaps make the result the inverse of the row-permuted matrix; its columns are
// permuted back at the end.  Work per matrix is one rank-GJ_NB product per panel instead
// of one pass over the whole matrix per column.
//
// A panel itself is treated the same way in strips of 16 columns and fewer: one block per matrix
// holds a strip of all rows in registers and eliminates it column by column (pivot search over
// the rows not yet pivoted, swap, elimination; two barriers a column), the strip's swaps go to the
// rest of the rows, and the panel's other columns receive a product of the strip's rank.  What
// bounds it is the chain of columns, about 2 us each, against four launches a column.  FP64:
// sixteen matrices of 192 columns 2.6 -> 0.75 ms, one of 1572 22.4 -> 8.0 ms, one of 5800 119 -> 79
// ms, of which 22 are the rank-64 products.
#include "kernels.h"

namespace thm {

constexpr int GJ_NB = 64;

__device__ __forceinline__ int find_sys2(const int32_t *blkoff, int nd, int b) {
    return blkoff[nd + 1 + b];  // block -> matrix map stored after the offsets
}

// Columns of a strip: a thread holds at most 64 entries, and its rows grow with the matrix.  512
// threads: two waves a SIMD share the registers, and the work that every wave repeats (pivot,
// reciprocal, pivot row) is small against its rows.
__host__ constexpr int gj_width(int rows) {
    return rows <= 4 ? 16 : rows <= 8 ? 8 : rows <= 16 ? 4 : rows <= 32 ? 2 : 1;
}
constexpr int GJ_W = gj_width(1), GJ_THREADS = 512;

// Largest entry over the block: every thread brings its own candidate (v < 0: none).  Lanes and
// waves with the largest value are ordered by their number.
__device__ __forceinline__ void block_pivot(double &v, int &i, double *bv, int *bi) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    double m = v;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o, 64));
    if (lane == __ffsll((unsigned long long)__ballot(v == m)) - 1) {
        bv[wave] = m;
        bi[wave] = i;
    }
    __syncthreads();
    v = bv[0];
    i = bi[0];
    for (int q = 1; q < nw; ++q)
        if (bv[q] > v) {
            v = bv[q];
            i = bi[q];
        }
}

// Columns [c0, c0 + W) of every row: thread t holds the rows t, t + blockDim, ...  The current
// column is the first register of a row; the registers rotate by one a column, so that the loop
// stays rolled.
template <int R, int W>
__global__ void __launch_bounds__(GJ_THREADS) k_bgj_strip(const InvDesc *__restrict__ ds, int c0) {
    __shared__ double bv[2][GJ_THREADS / 64], prow[2][W], crow[2][W];
    __shared__ int bi[2][GJ_THREADS / 64];
    const InvDesc d = ds[blockIdx.x];
    const int n = d.n, t = threadIdx.x, nt = blockDim.x;
    if (c0 >= n) return;
    const int w = min(W, n - c0);
    // rows enter and leave through a wave's 64 x C tile in LDS: H lanes a row instead of one row a lane
    constexpr int C = W < 8 ? W : 8, H = 64 / C;
    __shared__ double tile[GJ_THREADS / 64][64][C + 1];
    const int lane = t & 63, wave = t >> 6, tr = lane / C, tc = lane % C;
    double a[R][W];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int j0 = 0; j0 < W; j0 += C) {
            double v[C];
#pragma unroll
            for (int q = 0; q < C; ++q) {
                const int i = r * nt + wave * 64 + q * H + tr, k = j0 + tc;
                v[q] = i < n && k < w ? d.A[(int64_t)i * n + c0 + k] : 0.0;
            }
#pragma unroll
            for (int q = 0; q < C; ++q) tile[wave][q * H + tr][tc] = v[q];
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int q = 0; q < C; ++q) a[r][j0 + q] = tile[wave][lane][q];
            __builtin_amdgcn_wave_barrier();
        }
    bool bad = false;
#pragma unroll 1
    for (int c = 0; c < w; ++c) {
        const int col = c0 + c, h = c & 1;
        double v = -1.0;
        int p = col;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int i = r * nt + t;
            const double x = fabs(a[r][0]);
            if (i >= col && i < n && x > v) {
                v = x;
                p = i;
            }
        }
        block_pivot(v, p, bv[h], bi[h]);
        bad |= !(v > 0.0) || !isfinite(v);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int i = r * nt + t;
            if (i == p)
#pragma unroll
                for (int j = 0; j < W; ++j) prow[h][j] = a[r][j];
            if (i == col)  // becomes the scaled pivot row: 0 + 1 pr
#pragma unroll
                for (int j = 0; j < W; ++j) {
                    crow[h][j] = a[r][j];
                    a[r][j] = 0.0;
                }
        }
        __syncthreads();
        const double pv = prow[h][0], ipv = pv != 0.0 ? 1.0 / pv : 0.0;
        double f[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int i = r * nt + t;
            if (i == p && p != col)
#pragma unroll
                for (int j = 0; j < W; ++j) a[r][j] = crow[h][j];
            f[r] = i == col ? -1.0 : a[r][0];
        }
#pragma unroll
        for (int j = 0; j < W; ++j) {
            const double pr = j == W - 1 ? ipv : prow[h][(j + 1) % W] * ipv;
#pragma unroll
            for (int r = 0; r < R; ++r) a[r][j] = (j == W - 1 ? 0.0 : a[r][(j + 1) % W]) - f[r] * pr;
        }
        if (t == 0) d.piv[col] = p;
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int j0 = 0; j0 < W; j0 += C) {
#pragma unroll
            for (int q = 0; q < C; ++q) tile[wave][lane][q] = a[r][j0 + q];
            __builtin_amdgcn_wave_barrier();
            const int j = j0 + tc, k = j + w < W ? j + w : j + w - W;  // column of register j after w rotations
#pragma unroll
            for (int q = 0; q < C; ++q) {
                const int i = r * nt + wave * 64 + q * H + tr;
                const double v = tile[wave][q * H + tr][tc];
                if (i < n && k < w) d.A[(int64_t)i * n + c0 + k] = v;
            }
            __builtin_amdgcn_wave_barrier();
        }
    if (t == 0 && bad) atomicOr(d.status, 1);
}

// A strip of one column in memory, for matrices of more rows than a block can hold.
__global__ void __launch_bounds__(GJ_THREADS) k_bgj_column(const InvDesc *__restrict__ ds, int col) {
    __shared__ double bv[GJ_THREADS / 64], prow, crow;
    __shared__ int bi[GJ_THREADS / 64];
    const InvDesc d = ds[blockIdx.x];
    const int n = d.n, t = threadIdx.x;
    if (col >= n) return;
    double v = -1.0;
    int p = col;
#pragma unroll 4
    for (int i = col + t; i < n; i += GJ_THREADS) {
        const double x = fabs(d.A[(int64_t)i * n + col]);
        if (x > v) {
            v = x;
            p = i;
        }
    }
    block_pivot(v, p, bv, bi);
    if (t == 0) {
        prow = d.A[(int64_t)p * n + col];
        crow = d.A[(int64_t)col * n + col];
        d.piv[col] = p;
        if (!(v > 0.0) || !isfinite(v)) atomicOr(d.status, 1);
    }
    __syncthreads();
    const double ipv = prow != 0.0 ? 1.0 / prow : 0.0;
#pragma unroll 4
    for (int i = t; i < n; i += GJ_THREADS) {
        const double f = i == p ? crow : d.A[(int64_t)i * n + col];
        d.A[(int64_t)i * n + col] = i == col ? ipv : 0.0 - f * ipv;
    }
}

// The row swaps of the strip [c0, c0 + w), composed, on every other column and on the row order
// (the second half of piv); the new rows of the strip inside the panel [kb, kb + GJ_NB) also go to
// scr (w x GJ_NB) for the panel's update.  Every wave composes them in its lanes: lane k stands
// for the k-th row of the strip, lane W + k for its pivot row, if that lies outside and is the
// first of its kind.
template <int W>
__global__ void __launch_bounds__(256) k_bgj_swap(const InvDesc *__restrict__ ds, int c0, int kb,
                                                  double *__restrict__ scr) {
    const InvDesc d = ds[blockIdx.y];
    const int n = d.n, t = threadIdx.x, lane = t & 63;
    if (c0 >= n || (int)blockIdx.x * 256 >= n) return;
    const int w = min(W, n - c0);
    const int p = d.piv[c0 + min(lane % W, w - 1)];
    const int row = lane < W ? c0 + min(lane, w - 1) : p;
    int slot = -1, src = lane;
#pragma unroll
    for (int k = 0; k < W; ++k)
        if (slot < 0 && __builtin_amdgcn_readlane(p, k) == p) slot = W + k;
    if (p < c0 + w) slot = p - c0;
#pragma unroll
    for (int i = 0; i < W; ++i) {
        if (i >= w) break;
        const int q = __builtin_amdgcn_readlane(slot, i);
        const int si = __builtin_amdgcn_readlane(src, i), sq = __builtin_amdgcn_readlane(src, q);
        src = lane == i ? sq : lane == q ? si : src;
    }
    if (blockIdx.x == 0 && t < 64) {
        int32_t *order = d.piv + n;
        const int o = order[__shfl(row, src, 64)];
        if (lane < 2 * W && src != lane) order[row] = o;
    }
    const int j = blockIdx.x * 256 + t;
    const bool live = j < n && (j < c0 || j >= c0 + w);
    double v[2 * W];
#pragma unroll
    for (int k = 0; k < 2 * W; ++k) {
        const int from = __builtin_amdgcn_readlane(src, k), r = __builtin_amdgcn_readlane(row, from);
        if (live && (k < w || from != k)) v[k] = d.A[(int64_t)r * n + j];
    }
#pragma unroll
    for (int k = 0; k < 2 * W; ++k) {
        const int from = __builtin_amdgcn_readlane(src, k), r = __builtin_amdgcn_readlane(row, k);
        if (live && from != k) d.A[(int64_t)r * n + j] = v[k];
        if (k < W && k < w && live && j >= kb && j < kb + GJ_NB)
            scr[((int64_t)blockIdx.y * W + k) * GJ_NB + j - kb] = v[k];
    }
}

// The strip's elimination on the panel's other columns: 64 rows a block, 4 x 4 entries a thread
template <int W>
__global__ void __launch_bounds__(256) k_bgj_panel(const InvDesc *__restrict__ ds, int c0, int kb,
                                                   const double *__restrict__ scr) {
    __shared__ double cs[64][W + 1], ys[W][GJ_NB];
    const InvDesc d = ds[blockIdx.y];
    const int n = d.n, i0 = blockIdx.x * 64, t = threadIdx.x;
    if (c0 >= n || i0 >= n) return;
    const int w = min(W, n - c0), pw = min(GJ_NB, n - kb);
    for (int e = t; e < 64 * W; e += 256) {
        const int i = e / W, k = e % W;
        cs[i][k] = i0 + i < n && k < w ? d.A[(int64_t)(i0 + i) * n + c0 + k] : 0.0;
    }
    for (int e = t; e < W * GJ_NB; e += 256) {
        const int k = e / GJ_NB, j = e % GJ_NB;
        const bool in = k < w && j < pw && (kb + j < c0 || kb + j >= c0 + w);
        ys[k][j] = in ? scr[((int64_t)blockIdx.y * W + k) * GJ_NB + j] : 0.0;
    }
    const int j0 = (t & 15) * 4, r0 = (t >> 4) * 4;
    double acc[4][4];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int i = i0 + r0 + r;
            const bool in = i < n && (i < c0 || i >= c0 + w) && j0 + q < pw;
            acc[r][q] = in ? d.A[(int64_t)i * n + kb + j0 + q] : 0.0;
        }
    __syncthreads();
#pragma unroll 4
    for (int k = 0; k < W; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[r][q] += cs[r0 + r][k] * ys[k][j0 + q];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int i = i0 + r0 + r, j = kb + j0 + q;
            if (i < n && j0 + q < pw && (j < c0 || j >= c0 + w)) d.A[(int64_t)i * n + j] = acc[r][q];
        }
}

// A[r, not c] = T (the product A[r, c] A[r, not c], staged in W) for the panel rows r
__global__ void __launch_bounds__(256) k_bgj_copyback(const InvDesc *__restrict__ ds, const int32_t *__restrict__ blkoff,
                                                      int nd, int kb) {
    const int di = find_sys2(blkoff, nd, blockIdx.x);
    const InvDesc d = ds[di];
    const int n = d.n;
    const int w = min(GJ_NB, n - kb);
    const int64_t e = (int64_t)(blockIdx.x - blkoff[di]) * 256 + threadIdx.x;
    if (w <= 0 || e >= (int64_t)w * n) return;
    const int r = (int)(e / n), j = (int)(e % n);
    if (j >= kb && j < kb + w) return;
    d.A[(int64_t)(kb + r) * n + j] = d.W[(int64_t)r * n + j];
}

// Row order (second half of piv): the identity to begin with; its inverse, in the first half, at the end
__global__ void __launch_bounds__(256) k_bgj_order(const InvDesc *__restrict__ ds, bool invert) {
    const InvDesc d = ds[blockIdx.y];
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= d.n) return;
    if (invert) d.piv[d.piv[d.n + i]] = i;
    else d.piv[d.n + i] = i;
}

__global__ void __launch_bounds__(256) k_bgj_perm_apply(const InvDesc *__restrict__ ds,
                                                        const int32_t *__restrict__ blkoff, int nd) {
    const int di = find_sys2(blkoff, nd, blockIdx.x);
    const InvDesc d = ds[di];
    const int n = d.n;
    const int nch = (n + 255) / 256;
    const int local = blockIdx.x - blkoff[di];
    const int i = local / nch;
    const int j = (local - i * nch) * 256 + threadIdx.x;
    if (i >= n || j >= n) return;
    d.out[(int64_t)i * d.ldo + j] = d.A[(int64_t)i * n + d.piv[j]];
}

void launch_invert_blocked(const std::vector<InvDesc> &d, hipStream_t st) {
    if (d.empty()) return;
    const int nd = (int)d.size();
    int nmax = 0;
    std::vector<int64_t> units_perm(nd), units_copy(nd);
    for (int i = 0; i < nd; ++i) {
        nmax = std::max(nmax, d[i].n);
        units_perm[i] = (int64_t)d[i].n * ((d[i].n + 255) / 256);
        units_copy[i] = (int64_t)d[i].n * GJ_NB;
    }
    DBuf<InvDesc> dd;
    dd.upload(d, st);
    DBuf<double> scr((int64_t)nd * GJ_W * GJ_NB);
    Sched sperm, scopy;
    scopy.build(units_copy, 256, st);
    sperm.build(units_perm, 1, st);
    DBuf<GemmDesc> gscr;
    Sched gsched;
    const int threads = std::min(GJ_THREADS, (nmax + 63) / 64 * 64), rows = (nmax + threads - 1) / threads;
    const int width = gj_width(rows);
    const dim3 by_col((unsigned)((nmax + 255) / 256), nd), by_row((unsigned)((nmax + 63) / 64), nd);
    k_bgj_order<<<by_col, 256, 0, st>>>(dd.p, false);
    for (int kb = 0; kb < nmax; kb += GJ_NB) {
        const int kend = std::min(nmax, kb + GJ_NB);
        for (int c0 = kb; c0 < kend; c0 += width) {
            auto strip = [&](auto rc) {
                constexpr int R = decltype(rc)::value, W = gj_width(R);
                if constexpr (W > 1) k_bgj_strip<R, W><<<nd, threads, 0, st>>>(dd.p, c0);
                else k_bgj_column<<<nd, GJ_THREADS, 0, st>>>(dd.p, c0);
                k_bgj_swap<W><<<by_col, 256, 0, st>>>(dd.p, c0, kb, scr.p);
                k_bgj_panel<W><<<by_row, 256, 0, st>>>(dd.p, c0, kb, scr.p);
            };
            if (rows == 1) strip(std::integral_constant<int, 1>{});
            else if (rows == 2) strip(std::integral_constant<int, 2>{});
            else if (rows <= 4) strip(std::integral_constant<int, 4>{});
            else if (rows <= 8) strip(std::integral_constant<int, 8>{});
            else if (rows <= 16) strip(std::integral_constant<int, 16>{});
            else if (rows <= 32) strip(std::integral_constant<int, 32>{});
            else strip(std::integral_constant<int, 33>{});
        }
        THM_HIP(hipGetLastError());
        // rank-w updates of the columns outside the panel
        std::vector<GemmDesc> g;
        for (int i = 0; i < nd; ++i) {
            const int n = d[i].n;
            if (kb >= n) continue;
            const int w = std::min(GJ_NB, n - kb);
            const int lo[2] = {0, kb + w}, len[2] = {kb, n - kb - w};
            double *A = d[i].A;
            for (int a = 0; a < 2; ++a)
                for (int b = 0; b < 2; ++b) {
                    if (!len[a] || !len[b]) continue;
                    // A[I, J] += A[I, panel] A[panel, J]
                    g.push_back({len[a], len[b], w, 0, 0, A + (int64_t)lo[a] * n + kb, A + (int64_t)kb * n + lo[b],
                                 A + (int64_t)lo[a] * n + lo[b], n, n, n, 1.0, 1.0});
                }
            for (int b = 0; b < 2; ++b) {
                if (!len[b]) continue;
                // W[0:w, J] = A[panel, panel] A[panel, J]
                g.push_back({w, len[b], w, 0, 0, A + (int64_t)kb * n + kb, A + (int64_t)kb * n + lo[b],
                             d[i].W + lo[b], n, n, n, 1.0, 0.0});
            }
        }
        launch_gemm_batched(g, st, gscr, gsched);
        k_bgj_copyback<<<scopy.nblocks, 256, 0, st>>>(dd.p, scopy.blkoff.p, nd, kb);
        THM_HIP(hipGetLastError());
    }
    k_bgj_order<<<by_col, 256, 0, st>>>(dd.p, true);
    k_bgj_perm_apply<<<sperm.nblocks, 256, 0, st>>>(dd.p, sperm.blkoff.p, nd);
    THM_HIP(hipGetLastError());
    THM_HIP(hipStreamSynchronize(st));  // keeps the schedules and scratch alive until the kernels finished
}

}  // namespace thm
