// Linear-algebra kernels for gfx950: block SpMV on [[K,-C],[C,K]], Krylov vector
// operations (classical Gram-Schmidt with wave64 reductions, Givens in FP64),
// dense batched GEMM and Gauss-Jordan inversion (preconditioner setup), and the
// block-tridiagonal + static-condensation application of diag(K,K)^{-1}.
//
// Batching: every kernel serves several independent systems.  A flattened block
// schedule maps blockIdx.x to (system, block-in-system) so that systems of very
// different size share one launch without empty blocks.  Vectors of all systems
// live in one arena; system s owns scalars [off[s], off[s] + 2 n_s) of a slot,
// stored as interleaved (re, im) pairs.
#include "kernels.h"

namespace thm {

// ------------------------------------------------------------------ helpers
__device__ __forceinline__ int find_sys(const int32_t *blkoff, int ns, int b) {
    return blkoff[ns + 1 + b];  // block -> system map stored after the offsets
}

template <class T>
__device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Block reduction of one double over 256 threads (4 waves); result valid in thread 0.
__device__ __forceinline__ double block_sum256(double v, double *lds) {
    v = wave_sum(v);
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    __syncthreads();
    if (l == 0) lds[w] = v;
    __syncthreads();
    double r = 0.0;
    if (threadIdx.x == 0) r = lds[0] + lds[1] + lds[2] + lds[3];
    return r;
}

template <class T> struct V2;
template <> struct V2<double> { using t = double2; };
template <> struct V2<float> { using t = float2; };

// ------------------------------------------------------------------ SpMV
// y = A x  or  y = b - A x, A = [[K, -sC], [sC, K]] acting on interleaved (re, im)
// pairs, s = +1 (A) or -1 (A^T).  K is read once for both halves.  LPR lanes per row.
template <int LPR, int UNR, class T>
__global__ void __launch_bounds__(256) k_spmv(const MatDesc *__restrict__ mats, const int64_t *__restrict__ off,
                                              const int32_t *__restrict__ blkoff, int ns,
                                              const int32_t *__restrict__ mask, const T *__restrict__ xb,
                                              T *__restrict__ yb, const T *__restrict__ bb, float csign) {
    using T2 = typename V2<T>::t;
    const int s = find_sys(blkoff, ns, blockIdx.x);
    if (mask && !mask[s]) return;
    const MatDesc m = mats[s];
    constexpr int RPB = 256 / LPR;
    const int64_t row = (int64_t)(blockIdx.x - blkoff[s]) * RPB + threadIdx.x / LPR;
    const int lane = threadIdx.x % LPR;
    if (row >= m.n) return;
    const T2 *x = reinterpret_cast<const T2 *>(xb + off[s]);
    const T *kv = reinterpret_cast<const T *>(m.kval);
    T ar = 0, ai = 0;
    const int32_t r0 = m.rowptr[row], r1 = m.rowptr[row + 1];
    // UNR entries per lane are loaded before the FMAs (memory-level parallelism).
    int32_t q = r0 + lane;
    if (UNR > 1)
        for (; q + (UNR - 1) * LPR < r1; q += UNR * LPR) {
            T k[UNR];
            int32_t c[UNR];
#pragma unroll
            for (int u = 0; u < UNR; ++u) {
                k[u] = kv[q + u * LPR];
                c[u] = m.col[q + u * LPR];
            }
            T2 xv[UNR];
#pragma unroll
            for (int u = 0; u < UNR; ++u) xv[u] = x[c[u]];
#pragma unroll
            for (int u = 0; u < UNR; ++u) {
                ar += k[u] * xv[u].x;
                ai += k[u] * xv[u].y;
            }
        }
    for (; q < r1; q += LPR) {
        const T k = kv[q];
        const T2 xv = x[m.col[q]];
        ar += k * xv.x;
        ai += k * xv.y;
    }
#pragma unroll
    for (int o = LPR / 2; o > 0; o >>= 1) {
        ar += __shfl_xor(ar, o, LPR);
        ai += __shfl_xor(ai, o, LPR);
    }
    if (lane == 0) {
        const T *cv = reinterpret_cast<const T *>(m.cval);
        const T sg = (T)csign;
        for (int32_t q = m.crowptr[row]; q < m.crowptr[row + 1]; ++q) {
            const T c = sg * cv[q];
            const T2 xv = x[m.ccol[q]];
            ar -= c * xv.y;
            ai += c * xv.x;
        }
        T2 *y = reinterpret_cast<T2 *>(yb + off[s]);
        if (bb) {
            const T2 bv = reinterpret_cast<const T2 *>(bb + off[s])[row];
            y[row] = T2{bv.x - ar, bv.y - ai};
        } else {
            y[row] = T2{ar, ai};
        }
    }
}

// SELL-64 variant: one wave per slice of 64 (length-sorted) rows, one row per lane.  The value and
// column loads of a wave are 64 consecutive entries (coalesced), there is no cross-lane
// reduction and no divergence inside the K loop; padding entries have value 0 and point
// at a valid column.  The boundary operator C (few rows) is applied from its CSR.
template <class T>
__global__ void __launch_bounds__(256) k_spmv_sell(const MatDesc *__restrict__ mats, const int64_t *__restrict__ off,
                                                   const int32_t *__restrict__ blkoff, int ns,
                                                   const int32_t *__restrict__ mask, const T *__restrict__ xb,
                                                   T *__restrict__ yb, const T *__restrict__ bb, float csign) {
    using T2 = typename V2<T>::t;
    const int s = find_sys(blkoff, ns, blockIdx.x);
    if (mask && !mask[s]) return;
    const MatDesc &m = mats[s];
    const int64_t slice = (int64_t)(blockIdx.x - blkoff[s]) * 4 + (threadIdx.x >> 6);
    if (slice * SELL_C >= m.n) return;  // whole wave
    const int lane = threadIdx.x & 63;
    // the matrix (values, columns, row map) and y are touched once per call: non-temporal
    // loads and stores keep them from evicting the gathered entries of x from the caches
    const int32_t row = __builtin_nontemporal_load(m.sl_row + slice * SELL_C + lane);
    const T2 *x = reinterpret_cast<const T2 *>(xb + off[s]);
    const int32_t e0 = m.sl_ptr[slice], w = (m.sl_ptr[slice + 1] - e0) / SELL_C;
    const int32_t *cp = m.sl_col + e0 + lane;
    const T *vp = reinterpret_cast<const T *>(m.sl_val) + e0 + lane;
    T ar = 0, ai = 0;
    int k = 0;
    for (; k + 8 <= w; k += 8) {
        int32_t c[8];
        T v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            c[u] = __builtin_nontemporal_load(cp + (k + u) * SELL_C);
            v[u] = __builtin_nontemporal_load(vp + (k + u) * SELL_C);
        }
        T2 xv[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) xv[u] = x[c[u]];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            ar += v[u] * xv[u].x;
            ai += v[u] * xv[u].y;
        }
    }
    for (; k < w; ++k) {
        const T v = __builtin_nontemporal_load(vp + k * SELL_C);
        const T2 xv = x[__builtin_nontemporal_load(cp + k * SELL_C)];
        ar += v * xv.x;
        ai += v * xv.y;
    }
    if (row < 0) return;
    const T *cv = reinterpret_cast<const T *>(m.cval);
    const T sg = (T)csign;
    for (int32_t q = m.crowptr[row]; q < m.crowptr[row + 1]; ++q) {
        const T c = sg * cv[q];
        const T2 xv = x[m.ccol[q]];
        ar -= c * xv.y;
        ai += c * xv.x;
    }
    T2 *y = reinterpret_cast<T2 *>(yb + off[s]);
    if (bb) {
        const T2 bv = reinterpret_cast<const T2 *>(bb + off[s])[row];
        ar = bv.x - ar;
        ai = bv.y - ai;
    }
    __builtin_nontemporal_store(ar, &y[row].x);
    __builtin_nontemporal_store(ai, &y[row].y);
}

__global__ void __launch_bounds__(256) k_sell_fill(int64_t ne, const int32_t *__restrict__ src,
                                                   const double *__restrict__ kval, double *__restrict__ v64,
                                                   float *__restrict__ v32) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= ne) return;
    const double v = src[e] >= 0 ? kval[src[e]] : 0.0;
    v64[e] = v;
    v32[e] = (float)v;
}

void launch_sell_fill(int64_t ne, const int32_t *src, const double *kval, double *v64, float *v32, hipStream_t st) {
    if (ne <= 0) return;
    k_sell_fill<<<(unsigned)((ne + 255) / 256), 256, 0, st>>>(ne, src, kval, v64, v32);
    THM_HIP(hipGetLastError());
}

// Variant code v = 10 * lanes_per_row + unroll (unroll 1 or 4), or SPMV_SELL; chosen by
// the autotuner.
template <class T>
void launch_spmv(int v, const MatDesc *mats, const int64_t *off, const Sched &sc, int ns, const int32_t *mask,
                 const T *x, T *y, const T *b, float csign, hipStream_t st) {
    if (!sc.nblocks) return;
    const dim3 g(sc.nblocks), blk(256);
#define SPMV_CASE(L, U) \
    case 10 * L + U: k_spmv<L, U, T><<<g, blk, 0, st>>>(mats, off, sc.blkoff.p, ns, mask, x, y, b, csign); break;
    if (v == SPMV_SELL) {
        k_spmv_sell<T><<<g, blk, 0, st>>>(mats, off, sc.blkoff.p, ns, mask, x, y, b, csign);
        THM_HIP(hipGetLastError());
        return;
    }
    switch (v) {
        SPMV_CASE(2, 1) SPMV_CASE(4, 1) SPMV_CASE(8, 1) SPMV_CASE(16, 1) SPMV_CASE(32, 1) SPMV_CASE(64, 1)
        SPMV_CASE(2, 4) SPMV_CASE(4, 4) SPMV_CASE(8, 4) SPMV_CASE(16, 4) SPMV_CASE(32, 4)
        default: fail(THM_EINVAL, "unknown SpMV variant");
    }
#undef SPMV_CASE
    THM_HIP(hipGetLastError());
}
template void launch_spmv<double>(int, const MatDesc *, const int64_t *, const Sched &, int, const int32_t *,
                                  const double *, double *, const double *, float, hipStream_t);
template void launch_spmv<float>(int, const MatDesc *, const int64_t *, const Sched &, int, const int32_t *,
                                 const float *, float *, const float *, float, hipStream_t);

// Grouped SELL-64 variant: the systems of a group have the same K (pattern and values).
// A slice of 64 rows is served by up to four waves of one block, each applying it to four
// members' vectors (the group's count padded to a multiple of 4; the padding repeats the
// last member and is not stored), so K goes from HBM once per slice and its re-reads by
// the sibling waves hit the caches.  The sum over a row runs in the same order as in
// k_spmv_sell, so both variants give the same bits.  Each member's boundary operator C is
// applied from its own CSR, on the rows where some member has C entries.
// The four members' values of one x entry.  Per-member vectors (IL = false): four gathers.
// Member-interleaved copy (IL = true): the four values are one contiguous 4-complex run.
template <class T, bool IL>
struct GroupX;
template <class T>
struct GroupX<T, false> {
    using T2 = typename V2<T>::t;
    const T2 *x[4];
    __device__ __forceinline__ GroupX(const SpmvGroup &G, int j0, int nmw, const int64_t *off, const T *xb) {
#pragma unroll
        for (int j = 0; j < 4; ++j) x[j] = reinterpret_cast<const T2 *>(xb + off[G.mem[j0 + min(j, nmw - 1)]]);
    }
    __device__ __forceinline__ void load(int32_t c, T2 (&v)[4]) const {
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = x[j][c];
    }
    __device__ __forceinline__ T2 load1(int32_t c, int j) const { return x[j][c]; }
};
template <class T>
struct GroupX<T, true> {
    using T2 = typename V2<T>::t;
    typedef T vec4 __attribute__((ext_vector_type(4)));
    const T *x;
    int64_t ld;  // scalars per row of the interleaved copy
    __device__ __forceinline__ GroupX(const SpmvGroup &G, int j0, int, const int64_t *, const T *xib)
        : x(xib + 2 * (G.xoff + j0)), ld(2 * (int64_t)G.npad) {}
    __device__ __forceinline__ void load(int32_t c, T2 (&v)[4]) const {
        // 8 scalars of members j0 .. j0 + 3 (16-byte aligned: npad, j0 and xoff are multiples of 4)
        const vec4 *p = reinterpret_cast<const vec4 *>(x + c * ld);
        const vec4 a = p[0], b = p[1];
        v[0] = T2{a[0], a[1]};
        v[1] = T2{a[2], a[3]};
        v[2] = T2{b[0], b[1]};
        v[3] = T2{b[2], b[3]};
    }
    __device__ __forceinline__ T2 load1(int32_t c, int j) const {
        return reinterpret_cast<const T2 *>(x + c * ld)[j];
    }
};

template <class T, int U, bool IL>
__device__ __forceinline__ void spmv_group_slice(const MatDesc *__restrict__ mats, const int64_t *__restrict__ off,
                                                 const SpmvGroup &G, int j0, const MatDesc &m, int64_t slice,
                                                 const int32_t *__restrict__ mask, const T *__restrict__ xb,
                                                 T *__restrict__ yb, const T *__restrict__ bb, float csign) {
    using T2 = typename V2<T>::t;
    constexpr int MB = 4;
    const int nmw = min(MB, G.nm - j0);  // members of this wave (1 .. 4)
    const int lane = threadIdx.x & 63;
    const int32_t row = __builtin_nontemporal_load(m.sl_row + slice * SELL_C + lane);
    const int32_t e0 = m.sl_ptr[slice], w = (m.sl_ptr[slice + 1] - e0) / SELL_C;
    const int32_t *cp = m.sl_col + e0 + lane;
    const T *vp = reinterpret_cast<const T *>(m.sl_val) + e0 + lane;
    const GroupX<T, IL> x(G, j0, nmw, off, xb);
    T ar[MB], ai[MB];
#pragma unroll
    for (int j = 0; j < MB; ++j) ar[j] = ai[j] = 0;
    int k = 0;
    for (; k + U <= w; k += U) {
        int32_t c[U];
        T v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            c[u] = cp[(k + u) * SELL_C];
            v[u] = vp[(k + u) * SELL_C];
        }
        T2 xv[U][MB];
#pragma unroll
        for (int u = 0; u < U; ++u) x.load(c[u], xv[u]);
#pragma unroll
        for (int j = 0; j < MB; ++j)
#pragma unroll
            for (int u = 0; u < U; ++u) {
                ar[j] += v[u] * xv[u][j].x;
                ai[j] += v[u] * xv[u][j].y;
            }
    }
    for (; k < w; ++k) {
        const T v = vp[k * SELL_C];
        const int32_t c = cp[k * SELL_C];
        T2 xv[MB];
        x.load(c, xv);
#pragma unroll
        for (int j = 0; j < MB; ++j) {
            ar[j] += v * xv[j].x;
            ai[j] += v * xv[j].y;
        }
    }
    if (row < 0) return;
    if (G.crow[row]) {
        const T sg = (T)csign;
#pragma unroll
        for (int j = 0; j < MB; ++j) {
            if (j >= nmw) break;
            const MatDesc &mj = mats[G.mem[j0 + j]];
            const T *cv = reinterpret_cast<const T *>(mj.cval);
            for (int32_t q = mj.crowptr[row]; q < mj.crowptr[row + 1]; ++q) {
                const T c = sg * cv[q];
                const T2 xq = x.load1(mj.ccol[q], j);
                ar[j] -= c * xq.y;
                ai[j] += c * xq.x;
            }
        }
    }
#pragma unroll
    for (int j = 0; j < MB; ++j) {
        if (j >= nmw) break;
        const int s = G.mem[j0 + j];
        if (mask && !mask[s]) continue;
        T a = ar[j], b = ai[j];
        if (bb) {
            const T2 bv = reinterpret_cast<const T2 *>(bb + off[s])[row];
            a = bv.x - a;
            b = bv.y - b;
        }
        T2 *y = reinterpret_cast<T2 *>(yb + off[s]);
        __builtin_nontemporal_store(a, &y[row].x);
        __builtin_nontemporal_store(b, &y[row].y);
    }
}

// Block schedule: npad / 4 consecutive waves per slice (see SpmvGroup).  IL: x is the
// member-interleaved copy (see SpmvGroup::xoff) instead of the per-system vectors.
template <class T, bool IL>
__global__ void __launch_bounds__(256) k_spmv_sell_group(const MatDesc *__restrict__ mats,
                                                         const int64_t *__restrict__ off,
                                                         const SpmvGroup *__restrict__ groups,
                                                         const int32_t *__restrict__ blkoff, int ng,
                                                         const int32_t *__restrict__ mask,
                                                         const T *__restrict__ xb, T *__restrict__ yb,
                                                         const T *__restrict__ bb, float csign) {
    const int g = find_sys(blkoff, ng, blockIdx.x);
    const SpmvGroup &G = groups[g];
    const int nmc = G.npad / 4;
    const int64_t gw = (int64_t)(blockIdx.x - blkoff[g]) * 4 + (threadIdx.x >> 6);
    const int64_t slice = gw / nmc;
    const int j0 = 4 * (int)(gw - slice * nmc);
    const MatDesc &m = mats[G.rep];
    if (slice * SELL_C >= m.n) return;  // whole wave
    if (mask) {
        int any = 0;
        for (int j = j0; j < min(j0 + 4, G.nm); ++j) any |= mask[G.mem[j]];
        if (!any) return;
    }
    constexpr int U = sizeof(T) == 4 ? 4 : 2;
    spmv_group_slice<T, U, IL>(mats, off, G, j0, m, slice, mask, xb, yb, bb, csign);
}

template <class T>
void launch_spmv_group(const MatDesc *mats, const int64_t *off, const SpmvGroup *groups, const Sched &sc, int ng,
                       const int32_t *mask, const T *x, T *y, const T *b, float csign, hipStream_t st) {
    if (!sc.nblocks) return;
    k_spmv_sell_group<T, false><<<sc.nblocks, 256, 0, st>>>(mats, off, groups, sc.blkoff.p, ng, mask, x, y, b, csign);
    THM_HIP(hipGetLastError());
}
template <class T>
void launch_spmv_group_i(const MatDesc *mats, const int64_t *off, const SpmvGroup *groups, const Sched &sc, int ng,
                         const int32_t *mask, const T *xi, T *y, float csign, hipStream_t st) {
    if (!sc.nblocks) return;
    k_spmv_sell_group<T, true><<<sc.nblocks, 256, 0, st>>>(mats, off, groups, sc.blkoff.p, ng, mask, xi, y, nullptr,
                                                           csign);
    THM_HIP(hipGetLastError());
}
template void launch_spmv_group_i<double>(const MatDesc *, const int64_t *, const SpmvGroup *, const Sched &, int,
                                          const int32_t *, const double *, double *, float, hipStream_t);
template void launch_spmv_group_i<float>(const MatDesc *, const int64_t *, const SpmvGroup *, const Sched &, int,
                                         const int32_t *, const float *, float *, float, hipStream_t);
template void launch_spmv_group<double>(const MatDesc *, const int64_t *, const SpmvGroup *, const Sched &, int,
                                        const int32_t *, const double *, double *, const double *, float,
                                        hipStream_t);
template void launch_spmv_group<float>(const MatDesc *, const int64_t *, const SpmvGroup *, const Sched &, int,
                                       const int32_t *, const float *, float *, const float *, float, hipStream_t);

// ------------------------------------------------------------------ Krylov vector kernels
// Vectors are interleaved (re, im) pairs.  With cplx = 1 the Arnoldi process uses
// complex scalars (h = <v, w> = sum conj(v) w; the Krylov space is invariant under
// multiplication by i, i.e. the complex GMRES of K + iC expressed on the real block
// vectors); with cplx = 0 it is the real GMRES of the 2N real block system (the
// imaginary part of every inner product is dropped).  Hessenberg, Givens and the
// least-squares solve are FP64 (complex storage in both modes).
// Elementwise kernels: a block owns VCHUNK scalars of one system; sums leave one partial per
// block.  The inner products of an Arnoldi step have their own split: a block owns dch[s] scalars
// (see DBLOCKS) and DCOLS basis columns.
constexpr int PPT = VCHUNK / 512;  // complex pairs per thread
constexpr int CG = 4;              // basis columns loaded together (lincomb)
constexpr int UG = 8;              // basis columns loaded together (Gram-Schmidt update)

// Loads stay unconditional (so the compiler keeps them all in flight): lanes past the
// end of a vector read its last element and their contribution is dropped.
__device__ __forceinline__ int64_t clampi(int64_t i, int64_t np) { return i < np ? i : np - 1; }

// Sum of a block's 256 values, left in thread 0's slot of the partials.
__device__ __forceinline__ void block_store(double v, double *dst) {
    __shared__ double lds[4];
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) *dst = (lds[0] + lds[1]) + (lds[2] + lds[3]);
}

// Sum of the partials [b0, b1), the same value in all 256 threads of every block that asks.
__device__ __forceinline__ double sum_partials(const double *part, int b0, int b1) {
    __shared__ double lds[4];
    double a = 0.0;
    for (int b = b0 + (int)threadIdx.x; b < b1; b += 256) a += part[b];
    a = wave_sum(a);
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = a;
    __syncthreads();
    const double r = (lds[0] + lds[1]) + (lds[2] + lds[3]);
    __syncthreads();
    return r;
}

// 16 bytes of a vector: one complex pair in FP64, two in FP32.
template <class T> struct Pack;
template <> struct Pack<double> {
    static constexpr int N = 1;
    typedef double vec __attribute__((ext_vector_type(2)));
};
template <> struct Pack<float> {
    static constexpr int N = 2;
    typedef float vec __attribute__((ext_vector_type(4)));
};

// Inner products of w with DCOLS basis columns over a block's part of a system.  Blocks per
// system and column group: a single block per chunk (all columns in turn) left most of the chip
// idle on small and middle-sized systems (128^2 degree 1, 25 columns on average, FP64: 24 us; as
// split here 16 us).  Slots hold a multiple of 64 scalars, so a 16-byte load never leaves them.
template <class T>
__global__ void __launch_bounds__(256) k_dots(const int64_t *__restrict__ off, const int64_t *__restrict__ len,
                                              const int32_t *__restrict__ dch, const int32_t *__restrict__ blkoff,
                                              int ns, const int32_t *__restrict__ mask,
                                              const int32_t *__restrict__ jcnt, const T *__restrict__ V, int64_t ld,
                                              const T *__restrict__ w, double *__restrict__ part, int maxcols,
                                              int cplx, int32_t *__restrict__ step_ctr) {
    using VT = typename Pack<T>::vec;
    constexpr int N = Pack<T>::N;
    __shared__ double red[4][2 * DCOLS];
    // the step counter of the cycle advances here: no other kernel of the step's rest reads the
    // old value
    if (step_ctr && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *step_ctr += 1;
    const int s = find_sys(blkoff, ns, blockIdx.x);
    if (!mask[s]) return;
    const int j = jcnt[s], c0 = DCOLS * blockIdx.y;
    if (c0 > j) return;
    const int64_t base = off[s], np = len[s] / 2, chunk = dch[s] / 2;
    const int64_t p0 = (int64_t)(blockIdx.x - blkoff[s]) * chunk, p1 = min(np, p0 + chunk);
    const T *vc[DCOLS];
#pragma unroll
    for (int u = 0; u < DCOLS; ++u) vc[u] = V + (int64_t)min(c0 + u, j) * ld + base;
    double v[2 * DCOLS];
#pragma unroll
    for (int u = 0; u < 2 * DCOLS; ++u) v[u] = 0.0;
    // two sets of loads in turn: one is in flight while the other is used
    VT a, an, c[DCOLS], cn[DCOLS];
    auto fetch = [&](int64_t i, VT &x, VT (&d)[DCOLS]) {
        x = *reinterpret_cast<const VT *>(w + base + 2 * i);
#pragma unroll
        for (int u = 0; u < DCOLS; ++u) d[u] = *reinterpret_cast<const VT *>(vc[u] + 2 * i);
    };
    int64_t i = p0 + N * (int)threadIdx.x;
    if (i < p1) fetch(i, a, c);
    for (; i < p1; i += 256 * N) {
        if (i + 256 * N < p1) fetch(i + 256 * N, an, cn);
#pragma unroll
        for (int q = 0; q < N; ++q) {
            const bool in = N == 1 || i + q < p1;  // padding may hold anything
            const double wr = in ? (double)a[2 * q] : 0.0, wi = in ? (double)a[2 * q + 1] : 0.0;
#pragma unroll
            for (int u = 0; u < DCOLS; ++u) {
                const double cr = in ? (double)c[u][2 * q] : 0.0, ci = in ? (double)c[u][2 * q + 1] : 0.0;
                v[2 * u] += cr * wr + ci * wi;
                v[2 * u + 1] += cr * wi - ci * wr;
            }
        }
        a = an;
#pragma unroll
        for (int u = 0; u < DCOLS; ++u) c[u] = cn[u];
    }
    // sums over the wave, halving the values a lane carries with each exchange: lane l ends up
    // with value l / 4
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    static_assert(DCOLS == 8, "four halvings leave one of 16 values per lane");
#pragma unroll
    for (int n = DCOLS, o = 32; n >= 1; n /= 2, o /= 2) {
        const bool up = lane & o;
#pragma unroll
        for (int k = 0; k < n; ++k) {
            const double keep = up ? v[n + k] : v[k], send = up ? v[k] : v[n + k];
            v[k] = keep + __shfl_xor(send, o, 64);
        }
    }
    double r = v[0];
    r += __shfl_xor(r, 2, 64);
    r += __shfl_xor(r, 1, 64);
    if ((lane & 3) == 0) red[wave][lane >> 2] = r;
    __syncthreads();
    const int t = threadIdx.x;
    if (t < 2 * DCOLS && c0 + t / 2 <= j) {
        const double q = (red[0][t] + red[1][t]) + (red[2][t] + red[3][t]);
        part[(int64_t)blockIdx.x * maxcols + 2 * c0 + t] = (t & 1) && !cplx ? 0.0 : q;
    }
}

// out[s][k] = sum of the partial slots of system s over its inner-product blocks.
__global__ void __launch_bounds__(256) k_reduce_cols(const int32_t *__restrict__ blkoff, int ns,
                                                     const int32_t *__restrict__ mask,
                                                     const int32_t *__restrict__ jcnt, const double *__restrict__ part,
                                                     int maxcols, double *__restrict__ out, int ldo, int accumulate) {
    __shared__ double red[8][32];
    const int s = blockIdx.x;
    if (s >= ns || (mask && !mask[s])) return;
    const int nc = 2 * (jcnt[s] + 1);
    if ((int)blockIdx.y * 32 >= nc) return;
    const int l = threadIdx.x & 31, r = threadIdx.x >> 5, c = blockIdx.y * 32 + l;  // 32 columns, 8 slot classes
    double acc = 0.0;
    if (c < nc)
#pragma unroll 4
        for (int b = blkoff[s] + r; b < blkoff[s + 1]; b += 8) acc += part[(int64_t)b * maxcols + c];
    red[r][l] = acc;
    __syncthreads();
    if (r || c >= nc) return;
#pragma unroll
    for (int q = 1; q < 8; ++q) acc += red[q][l];
    double *o = out + (int64_t)s * ldo + c;
    *o = accumulate ? *o + acc : acc;
}

// w -= sum_c V_c h_c (complex h), plus per-block partial ||w||^2.  h comes from hcol, or (fused)
// from the partials of the inner products: every block sums them itself, which replaces a launch
// where there are few of them (rule at launch_cgs_update); a system's first block then leaves the
// sums in hcol.  The first block also leaves the step's column and flag in jcol / actc, which
// the closing kernel reads while it changes jcnt and active.
template <class T>
__global__ void __launch_bounds__(256) k_cgs_update(const int64_t *__restrict__ off, const int64_t *__restrict__ len,
                                                    const int32_t *__restrict__ blkoff,
                                                    const int32_t *__restrict__ dblkoff, int ns,
                                                    const int32_t *__restrict__ mask, const int32_t *__restrict__ jcnt,
                                                    const T *__restrict__ V, int64_t ld, T *__restrict__ w,
                                                    double *__restrict__ h, int ldh, int fused,
                                                    const double *__restrict__ part, int maxcols,
                                                    double *__restrict__ npart, int32_t *__restrict__ jcol,
                                                    int32_t *__restrict__ actc) {
    using VT = typename Pack<T>::vec;
    constexpr int N = Pack<T>::N, R = VCHUNK / 2 / (256 * N);  // 16-byte loads per thread and column
    static_assert(R >= 1, "chunk too small");
    extern __shared__ double hs[];
    const int s = find_sys(blkoff, ns, blockIdx.x);
    const bool first = (int)blockIdx.x == blkoff[s];
    const bool on = mask[s];
    const int j = jcnt[s];
    if (first && threadIdx.x == 0) {
        jcol[s] = j;
        actc[s] = on;
    }
    if (!on) return;
    const int64_t base = off[s], np = len[s] / 2;
    const int64_t p0 = (int64_t)(blockIdx.x - blkoff[s]) * (VCHUNK / 2);
    double *hsys = h + (int64_t)s * ldh;
    for (int c = threadIdx.x; c < 2 * (j + 1); c += 256) {
        double a;
        if (fused) {
            a = 0.0;
#pragma unroll 8
            for (int b = dblkoff[s]; b < dblkoff[s + 1]; ++b) a += part[(int64_t)b * maxcols + c];
            if (first) hsys[c] = a;
        } else {
            a = hsys[c];
        }
        hs[c] = a;
    }
    // element r of this thread: pairs i .. i + N - 1; reads past the end stay inside the slot's
    // padding or at the last element
    int64_t at[R];
    double xr[R][N], xi[R][N];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t i = p0 + N * (r * 256 + (int64_t)threadIdx.x);
        at[r] = i < np ? i : (np - 1) / N * N;
        const VT v = *reinterpret_cast<const VT *>(w + base + 2 * at[r]);
#pragma unroll
        for (int q = 0; q < N; ++q) {
            xr[r][q] = v[2 * q];
            xi[r][q] = v[2 * q + 1];
        }
    }
    // two sets of columns in turn: one is in flight while the other is used
    VT v[UG][R], nx[UG][R];
    auto fetch = [&](int c0, VT (&d)[UG][R]) {
#pragma unroll
        for (int u = 0; u < UG; ++u) {
            const T *vc = V + (int64_t)min(c0 + u, j) * ld + base;
            // last read of the basis in this Arnoldi step (the next step streams the
            // preconditioner and the operator first): non-temporal
#pragma unroll
            for (int r = 0; r < R; ++r)
                d[u][r] = __builtin_nontemporal_load(reinterpret_cast<const VT *>(vc + 2 * at[r]));
        }
    };
    fetch(0, v);
    __syncthreads();
    for (int c0 = 0; c0 <= j; c0 += UG) {
        if (c0 + UG <= j) fetch(c0 + UG, nx);
#pragma unroll
        for (int u = 0; u < UG; ++u) {
            if (c0 + u > j) break;
            const double hr = hs[2 * (c0 + u)], hi = hs[2 * (c0 + u) + 1];
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int q = 0; q < N; ++q) {
                    xr[r][q] -= hr * (double)v[u][r][2 * q] - hi * (double)v[u][r][2 * q + 1];
                    xi[r][q] -= hr * (double)v[u][r][2 * q + 1] + hi * (double)v[u][r][2 * q];
                }
        }
#pragma unroll
        for (int u = 0; u < UG; ++u)
#pragma unroll
            for (int r = 0; r < R; ++r) v[u][r] = nx[u][r];
    }
    double nrm = 0.0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t i = p0 + N * (r * 256 + (int64_t)threadIdx.x);
#pragma unroll
        for (int q = 0; q < N; ++q) {
            if (i + q >= np) break;
            const T a = (T)xr[r][q], b = (T)xi[r][q];
            w[base + 2 * (i + q)] = a;
            w[base + 2 * (i + q) + 1] = b;
            nrm += (double)a * (double)a + (double)b * (double)b;
        }
    }
    block_store(nrm, npart + blockIdx.x);
}

// Per-block partials of ||x||^2.
template <class T>
__global__ void __launch_bounds__(256) k_norm2(const int64_t *__restrict__ off, const int64_t *__restrict__ len,
                                               const int32_t *__restrict__ blkoff, int ns,
                                               const int32_t *__restrict__ mask, const T *__restrict__ x,
                                               double *__restrict__ part) {
    const int s = find_sys(blkoff, ns, blockIdx.x);
    if (mask && !mask[s]) return;
    const int64_t base = off[s], n = len[s];
    const int64_t i0 = (int64_t)(blockIdx.x - blkoff[s]) * VCHUNK;
    double a = 0.0;
#pragma unroll
    for (int t = 0; t < VCHUNK / 256; ++t) {
        const int64_t i = i0 + t * 256 + threadIdx.x;
        const double v = (double)x[base + clampi(i, n)];
        a += i < n ? v * v : 0.0;
    }
    block_store(a, part + blockIdx.x);
}

// y = a_s * x (a_s = scal[s] or 1/scal[s]); optional second destination.
template <class TI, class TO>
__global__ void __launch_bounds__(256) k_scale(const int64_t *__restrict__ off, const int64_t *__restrict__ len,
                                               const int32_t *__restrict__ blkoff, int ns,
                                               const int32_t *__restrict__ mask, const double *__restrict__ scal,
                                               int invert, const TI *__restrict__ x, TO *__restrict__ y1,
                                               const int32_t *__restrict__ jcol, int64_t ld1, TO *__restrict__ y2) {
    const int s = find_sys(blkoff, ns, blockIdx.x);
    if (mask && !mask[s]) return;
    const int64_t base = off[s], n = len[s];
    const int64_t i0 = (int64_t)(blockIdx.x - blkoff[s]) * VCHUNK;
    double a = scal ? scal[s] : 1.0;
    if (invert) a = a != 0.0 ? 1.0 / a : 0.0;
    TO *d1 = y1 + base + (jcol ? (int64_t)jcol[s] * ld1 : 0);
#pragma unroll
    for (int t = 0; t < VCHUNK / 256; ++t) {
        const int64_t i = i0 + t * 256 + threadIdx.x;
        const TO v = (TO)(a * (double)x[base + clampi(i, n)]);
        if (i < n) {
            d1[i] = v;
            if (y2) y2[base + i] = v;
        }
    }
}

// y = sum_{c<k} V_c coef[s][c] (complex coefficients), k = kcnt[s].
template <class T>
__global__ void __launch_bounds__(256) k_lincomb(const int64_t *__restrict__ off, const int64_t *__restrict__ len,
                                                 const int32_t *__restrict__ blkoff, int ns,
                                                 const int32_t *__restrict__ mask, const int32_t *__restrict__ kcnt,
                                                 const T *__restrict__ V, int64_t ld, const double *__restrict__ coef,
                                                 int ldc, T *__restrict__ y) {
    using T2 = typename V2<T>::t;
    const int s = find_sys(blkoff, ns, blockIdx.x);
    if (mask && !mask[s]) return;
    const int k = kcnt[s];
    const int64_t base = off[s], np = len[s] / 2;
    const int64_t p0 = (int64_t)(blockIdx.x - blkoff[s]) * (VCHUNK / 2);
    double xr[PPT], xi[PPT];
#pragma unroll
    for (int t = 0; t < PPT; ++t) xr[t] = xi[t] = 0.0;
    for (int c0 = 0; c0 < k; c0 += CG) {
        T2 v[CG][PPT];
#pragma unroll
        for (int u = 0; u < CG; ++u) {
            const T2 *vc = reinterpret_cast<const T2 *>(V + (int64_t)min(c0 + u, k - 1) * ld + base);
#pragma unroll
            for (int t = 0; t < PPT; ++t) v[u][t] = vc[clampi(p0 + t * 256 + threadIdx.x, np)];
        }
#pragma unroll
        for (int u = 0; u < CG; ++u) {
            if (c0 + u >= k) break;
            const double ar = coef[(int64_t)s * ldc + 2 * (c0 + u)], ai = coef[(int64_t)s * ldc + 2 * (c0 + u) + 1];
#pragma unroll
            for (int t = 0; t < PPT; ++t) {
                xr[t] += ar * (double)v[u][t].x - ai * (double)v[u][t].y;
                xi[t] += ar * (double)v[u][t].y + ai * (double)v[u][t].x;
            }
        }
    }
    T2 *yp = reinterpret_cast<T2 *>(y + base);
#pragma unroll
    for (int t = 0; t < PPT; ++t) {
        const int64_t i = p0 + t * 256 + threadIdx.x;
        if (i < np) yp[i] = T2{(T)xr[t], (T)xi[t]};
    }
}

// x += a_s * z (a_s = scal ? scal[s] : 1), x in TX, z in TZ.
template <class TX, class TZ>
__global__ void __launch_bounds__(256) k_axpy(const int64_t *__restrict__ off, const int64_t *__restrict__ len,
                                              const int32_t *__restrict__ blkoff, int ns,
                                              const int32_t *__restrict__ mask, const double *__restrict__ scal,
                                              const TZ *__restrict__ z, TX *__restrict__ x) {
    const int s = find_sys(blkoff, ns, blockIdx.x);
    if (mask && !mask[s]) return;
    const int64_t base = off[s], n = len[s];
    const int64_t i0 = (int64_t)(blockIdx.x - blkoff[s]) * VCHUNK;
    const double a = scal ? scal[s] : 1.0;
#pragma unroll
    for (int t = 0; t < VCHUNK / 256; ++t) {
        const int64_t i = i0 + t * 256 + threadIdx.x;
        const int64_t ic = base + clampi(i, n);
        const TX v = (TX)((double)x[ic] + a * (double)z[ic]);
        if (i < n) x[base + i] = v;
    }
}

// Start of a GMRES cycle (one block of 256 per system): beta = ||r||; systems with
// beta/bnorm <= rtol stop; otherwise g = (beta, 0, ...), jcnt = 0, active = 1.  The
// tolerance is read from device memory (the launch may be replayed from a graph); the
// step counter of the cycle is reset; each system's running flag is also written to
// host-visible memory (hrun, may be null).  stepped (may be null) marks systems that took a first
// step: only those whose residual is not below resid0 keep the mark, and 2 is written for them.
__global__ void k_cycle_start(int ns, const int32_t *__restrict__ blkoff, const double *__restrict__ part,
                              int32_t *__restrict__ running, int32_t *__restrict__ active,
                              int32_t *__restrict__ jcnt, const double *__restrict__ bnorm,
                              const double *__restrict__ rtol_d, double *__restrict__ g, int m,
                              double *__restrict__ beta_out, double *__restrict__ resid_out,
                              int32_t *__restrict__ iters, int max_iter, int32_t *__restrict__ step_ctr,
                              int32_t *__restrict__ hrun, const double *__restrict__ resid0,
                              int32_t *__restrict__ stepped) {
    const int s = blockIdx.x;
    if (s >= ns) return;
    if (s == 0 && threadIdx.x == 0 && step_ctr) *step_ctr = 0;
    if (!running[s]) {
        if (threadIdx.x == 0) {
            active[s] = 0;
            if (hrun) hrun[s] = 0;
        }
        return;
    }
    const double rtol = *rtol_d;
    const double beta = sqrt(sum_partials(part, blkoff[s], blkoff[s + 1]));
    double *gs = g + (int64_t)s * 2 * (m + 1);
    for (int i = threadIdx.x; i < 2 * (m + 1); i += blockDim.x) gs[i] = 0.0;
    if (threadIdx.x != 0) return;
    const double rel = bnorm[s] > 0.0 ? beta / bnorm[s] : 0.0;
    resid_out[s] = rel;
    beta_out[s] = beta;
    jcnt[s] = 0;
    const bool undo = stepped && stepped[s] && !(rel < resid0[s]);
    if (stepped) stepped[s] = undo;
    if (!(rel > rtol) || iters[s] >= max_iter || !isfinite(rel)) {
        running[s] = 0;
        active[s] = 0;
        if (hrun) hrun[s] = undo ? 2 : 0;
        return;
    }
    active[s] = 1;
    if (hrun) hrun[s] = undo ? 2 : 1;
    gs[0] = beta;
}

// After Arnoldi step j of a system: h_{j+1,j} = ||w||, apply the previous complex Givens rotations
// to column j of H, build the new one, update g (one wave).
// Rotation G = [[c, s], [-conj(s), c]] with c real: G [a; b] = [r; 0].
// The rotated entry x_{i+1} = -conj(s_i) x_i + c_i h_{i+1} of one rotation enters the next: an
// affine recurrence, evaluated for 64 rotations at a time as a scan over the wave (six exchanges
// instead of a chain of 64 dependent steps; |s_i| <= 1, so the composed factors do not grow).
__device__ __forceinline__ void arnoldi_column(int s, int ns, double hn, const double *__restrict__ hcol, int ldh,
                                               double *__restrict__ H, double *__restrict__ cs,
                                               double *__restrict__ sn, double *__restrict__ g, int j,
                                               int32_t *__restrict__ active, int32_t *__restrict__ jcnt,
                                               double *__restrict__ hnext, const double *__restrict__ bnorm,
                                               const double *__restrict__ rtol_d, int m, int32_t *__restrict__ iters,
                                               int max_iter, double *__restrict__ resid_est, int32_t *__restrict__ hf) {
    const int lane = threadIdx.x & 63;
    double *gs = g + (int64_t)s * 2 * (m + 1);
    // read ahead of the scan
    const double gr = gs[2 * j], gi = gs[2 * j + 1], bn = bnorm[s], rtol = *rtol_d;
    const int it = iters[s] + 1;
    const double2 *hc = reinterpret_cast<const double2 *>(hcol + (int64_t)s * ldh);
    double *css = cs + (int64_t)s * m;
    double2 *sns = reinterpret_cast<double2 *>(sn + (int64_t)s * 2 * m);
    double2 *Hs = reinterpret_cast<double2 *>(H + (int64_t)s * 2 * (m + 1) * m) + (int64_t)j * (m + 1);
    double2 x = hc[0];  // entry i0 after the rotations before it
    for (int i0 = 0; i0 < j; i0 += 64) {
        const int i = i0 + lane;
        const bool in = i < j;
        const double c = in ? css[i] : 1.0;
        const double2 sv = in ? sns[i] : double2{0.0, 0.0};
        const double2 h1 = in ? hc[i + 1] : double2{0.0, 0.0};
        // affine map of this lane: x -> a x + b (identity past the end)
        double ar = in ? -sv.x : 1.0, ai = in ? sv.y : 0.0, br = c * h1.x, bi = c * h1.y;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const double pr = __shfl_up(ar, o, 64), pi = __shfl_up(ai, o, 64);
            const double qr = __shfl_up(br, o, 64), qi = __shfl_up(bi, o, 64);
            if (lane >= o) {
                br += ar * qr - ai * qi;
                bi += ar * qi + ai * qr;
                const double tr = ar * pr - ai * pi;
                ai = ar * pi + ai * pr;
                ar = tr;
            }
        }
        const double2 out{ar * x.x - ai * x.y + br, ar * x.y + ai * x.x + bi};  // x_{i+1}
        double2 xi{__shfl_up(out.x, 1, 64), __shfl_up(out.y, 1, 64)};
        if (lane == 0) xi = x;
        if (in) Hs[i] = double2{c * xi.x + (sv.x * h1.x - sv.y * h1.y), c * xi.y + (sv.x * h1.y + sv.y * h1.x)};
        x = double2{__shfl(out.x, 63, 64), __shfl(out.y, 63, 64)};
    }
    if (lane != 0) return;
    const double ar = x.x, ai = x.y;
    const double na = hypot(ar, ai), nb = fabs(hn);  // entry j + 1 of the column is real
    const double den = hypot(na, nb);
    double c = 1.0, sr = 0.0, si = 0.0, rr = ar, ri = ai;
    if (den > 0.0) {
        if (na == 0.0) {
            c = 0.0;  // rotation maps b to the top: [c a + s b] = b, -conj(s) a + c b = 0
            sr = 1.0;
            rr = hn;
            ri = 0.0;
        } else {
            const double ur = ar / na, ui = ai / na;  // a/|a|
            c = na / den;
            sr = ur * hn / den;  // s = (a/|a|) conj(b) / den
            si = ui * hn / den;
            rr = ur * den;
            ri = ui * den;
        }
    }
    css[j] = c;
    sns[j] = double2{sr, si};
    Hs[j] = double2{rr, ri};
    Hs[j + 1] = double2{0.0, 0.0};
    // g_{j+1} = -conj(s) g_j ; g_j = c g_j
    const double g1r = -(sr * gr + si * gi), g1i = -(sr * gi - si * gr);
    gs[2 * (j + 1)] = g1r;
    gs[2 * (j + 1) + 1] = g1i;
    gs[2 * j] = c * gr;
    gs[2 * j + 1] = c * gi;
    hnext[s] = hn;
    jcnt[s] = j + 1;
    iters[s] = it;
    const double est = hypot(g1r, g1i) / bn;
    resid_est[s] = est;
    const bool breakdown = !(hn > 1e-300) || !(den > 0.0);
    const int32_t on = !(est <= rtol || breakdown || j + 1 >= m || it >= max_iter || !isfinite(est));
    active[s] = on;
    *hf = on;
}

// Close of an Arnoldi step, one launch: V_{j+1} = cur = w / ||w|| on the vector blocks, and the
// column of H (arnoldi_column) on one more block per system.  The vector blocks read the step's
// column and flag from jcol / actc, since the column blocks change jcnt and active meanwhile.
// hflags: one slot per group of spc consecutive steps, the last step of the group leaves its
// flag there (step_ctr counts this step already).
template <class T>
__global__ void __launch_bounds__(256) k_arnoldi_close(
    const int64_t *__restrict__ off, const int64_t *__restrict__ len, const int32_t *__restrict__ blkoff, int nvb,
    int ns, const double *__restrict__ npart, const int32_t *__restrict__ jcol, const int32_t *__restrict__ actc,
    const T *__restrict__ w, T *__restrict__ V, int64_t ld, T *__restrict__ cur, const double *__restrict__ hcol,
    int ldh, double *__restrict__ H, double *__restrict__ cs, double *__restrict__ sn, double *__restrict__ g,
    int32_t *__restrict__ active, int32_t *__restrict__ jcnt, double *__restrict__ hnext,
    const double *__restrict__ bnorm, const double *__restrict__ rtol_d, int m, int32_t *__restrict__ iters,
    int max_iter, double *__restrict__ resid_est, int32_t *__restrict__ hflags, const int32_t *__restrict__ step_ctr,
    int spc, int nslots) {
    const bool column = (int)blockIdx.x < ns;  // the column blocks first: theirs is the longer chain
    const int vb = (int)blockIdx.x - ns;
    const int s = column ? (int)blockIdx.x : find_sys(blkoff, ns, vb);
    int32_t *hf = hflags + (int64_t)(((*step_ctr - 1) / spc) % nslots) * ns + s;
    if (!actc[s]) {
        if (column && threadIdx.x == 0) *hf = 0;
        return;
    }
    const int j = jcol[s];
    const double hn = sqrt(sum_partials(npart, blkoff[s], blkoff[s + 1]));
    if (column) {
        if (threadIdx.x < 64)
            arnoldi_column(s, ns, hn, hcol, ldh, H, cs, sn, g, j, active, jcnt, hnext, bnorm, rtol_d, m, iters,
                           max_iter, resid_est, hf);
        return;
    }
    const double a = hn != 0.0 ? 1.0 / hn : 0.0;
    const int64_t base = off[s], n = len[s];
    const int64_t i0 = (int64_t)(vb - blkoff[s]) * VCHUNK;
    T *d = V + base + (int64_t)(j + 1) * ld;
#pragma unroll
    for (int t = 0; t < VCHUNK / 512; ++t) {
        const int64_t i = i0 + 2 * (t * 256 + (int64_t)threadIdx.x);  // a complex pair
        if (i >= n) break;
        using T2 = typename V2<T>::t;
        const T2 x = *reinterpret_cast<const T2 *>(w + base + i);
        const T2 v{(T)(a * (double)x.x), (T)(a * (double)x.y)};
        *reinterpret_cast<T2 *>(d + i) = v;
        *reinterpret_cast<T2 *>(cur + base + i) = v;
    }
}

// y = H^{-1} g on the first k = jcnt[s] columns (upper triangular, complex); one wave
// per system, column-oriented back substitution.
__global__ void k_hsolve(int ns, const int32_t *__restrict__ running, const int32_t *__restrict__ jcnt,
                         const double *__restrict__ H, const double *__restrict__ g, double *__restrict__ y, int m) {
    __shared__ double rr[1025], ri[1025];
    const int s = blockIdx.x;
    if (s >= ns || !running[s]) return;
    const int k = jcnt[s];
    const double *Hs = H + (int64_t)s * 2 * (m + 1) * m;
    const double *gs = g + (int64_t)s * 2 * (m + 1);
    double *ys = y + (int64_t)s * 2 * (m + 1);
    for (int i = threadIdx.x; i < k; i += blockDim.x) {
        rr[i] = gs[2 * i];
        ri[i] = gs[2 * i + 1];
    }
    __syncthreads();
    for (int i = k - 1; i >= 0; --i) {
        const double *col = Hs + (int64_t)i * 2 * (m + 1);
        const double dr = col[2 * i], di = col[2 * i + 1];
        const double den = dr * dr + di * di;
        // y_i = r_i / d
        const double yr = den > 0.0 ? (rr[i] * dr + ri[i] * di) / den : 0.0;
        const double yi = den > 0.0 ? (ri[i] * dr - rr[i] * di) / den : 0.0;
        for (int r = threadIdx.x; r < i; r += blockDim.x) {
            const double hr = col[2 * r], hi = col[2 * r + 1];
            rr[r] -= hr * yr - hi * yi;
            ri[r] -= hr * yi + hi * yr;
        }
        if (threadIdx.x == 0) {
            ys[2 * i] = yr;
            ys[2 * i + 1] = yi;
        }
        __syncthreads();
    }
}

__global__ void k_solve_reset(int ns, const int32_t *__restrict__ mask, int32_t *__restrict__ running,
                              int32_t *__restrict__ iters) {
    const int s = blockIdx.x * 256 + threadIdx.x;
    if (s >= ns) return;
    running[s] = mask[s];
    iters[s] = 0;
}
// Counts the first step of the running systems, marks them and keeps their residuals before it.
__global__ void k_first_step(int ns, const int32_t *__restrict__ running, int32_t *__restrict__ iters,
                             const double *__restrict__ resid, double *__restrict__ resid0,
                             int32_t *__restrict__ stepped) {
    const int s = blockIdx.x * 256 + threadIdx.x;
    if (s >= ns) return;
    stepped[s] = running[s];
    if (!running[s]) return;
    iters[s] += 1;
    resid0[s] = resid[s];
}
// Per system an integer and up to two numbers for the host, in its own memory.
__global__ void k_export(int ns, const int32_t *__restrict__ n, const double *__restrict__ a,
                         const double *__restrict__ b, double *__restrict__ out) {
    const int s = blockIdx.x * 256 + threadIdx.x;
    if (s >= ns) return;
    out[3 * s] = n[s];
    if (a) out[3 * s + 1] = a[s];
    if (b) out[3 * s + 2] = b[s];
}
// Of one system: the column count, the residual estimate and the newest column of H.
__global__ void k_export_column(const int32_t *__restrict__ jcnt, const double *__restrict__ est,
                                const double *__restrict__ H, int m, double *__restrict__ out) {
    const int j = *jcnt;
    if (threadIdx.x == 0) {
        out[0] = j;
        out[1] = *est;
    }
    for (int i = threadIdx.x; i < 2 * j; i += 256) out[2 + i] = H[(int64_t)(j - 1) * 2 * (m + 1) + i];
}
void launch_solve_reset(const Batch &B, const int32_t *mask, int32_t *running, int32_t *iters, hipStream_t st) {
    k_solve_reset<<<(B.ns + 255) / 256, 256, 0, st>>>(B.ns, mask, running, iters);
    THM_HIP(hipGetLastError());
}
void launch_first_step(const Batch &B, const int32_t *running, int32_t *iters, const double *resid, double *resid0,
                       int32_t *stepped, hipStream_t st) {
    k_first_step<<<(B.ns + 255) / 256, 256, 0, st>>>(B.ns, running, iters, resid, resid0, stepped);
    THM_HIP(hipGetLastError());
}
void launch_export(const Batch &B, const int32_t *n, const double *a, const double *b, double *out, hipStream_t st) {
    k_export<<<(B.ns + 255) / 256, 256, 0, st>>>(B.ns, n, a, b, out);
    THM_HIP(hipGetLastError());
}
void launch_export_column(const int32_t *jcnt, const double *est, const double *H, int m, double *out, hipStream_t st) {
    k_export_column<<<1, 256, 0, st>>>(jcnt, est, H, m, out);
    THM_HIP(hipGetLastError());
}

// Zero the entries flagged in `dir` (Dirichlet rows) of a complex vector.
template <class T>
__global__ void k_zero_flagged(const int64_t *__restrict__ off, const int64_t *__restrict__ nvec,
                               const int32_t *__restrict__ blkoff, int ns, const uint8_t *const *__restrict__ dirs,
                               T *__restrict__ x) {
    const int s = find_sys(blkoff, ns, blockIdx.x);
    const int64_t i = (int64_t)(blockIdx.x - blkoff[s]) * 256 + threadIdx.x;
    if (i >= nvec[s]) return;
    if (dirs[s][i]) { x[off[s] + 2 * i] = (T)0; x[off[s] + 2 * i + 1] = (T)0; }
}

// out[s] = sqrt(sum of partials); with bnorm: resid[s] = out/bnorm, running[s] = 0 if <= rtol.
__global__ void k_norm_finish(int ns, const int32_t *__restrict__ blkoff, const double *__restrict__ part,
                              const int32_t *__restrict__ mask, double *__restrict__ out,
                              const double *__restrict__ bnorm, double rtol, double *__restrict__ resid,
                              int32_t *__restrict__ running) {
    const int s = blockIdx.x;
    if (s >= ns || (mask && !mask[s])) return;
    const double nrm = sqrt(sum_partials(part, blkoff[s], blkoff[s + 1]));
    if (threadIdx.x != 0) return;
    out[s] = nrm;
    if (bnorm) {
        const double rel = bnorm[s] > 0.0 ? nrm / bnorm[s] : 0.0;
        resid[s] = rel;
        if (running && !(rel > rtol)) running[s] = 0;
    }
}

// ------------------------------------------------------------------ launchers
#define VGRID(sc) dim3((sc).nblocks), dim3(256), 0, st
#define VGUARD(B) if (!(B).vs.nblocks) return

template <class T>
void launch_dots(const Batch &B, const int32_t *mask, const int32_t *jcnt, const T *V, int64_t ld, const T *w,
                 double *part, int cplx, int32_t *step_ctr, hipStream_t st) {
    VGUARD(B);
    const dim3 grid(B.ds.nblocks, (B.maxcols / 2 + DCOLS - 1) / DCOLS);
    k_dots<T><<<grid, 256, 0, st>>>(B.off.p, B.len.p, B.dch.p, B.ds.blkoff.p, B.ns, mask, jcnt, V, ld, w, part,
                                    B.maxcols, cplx, step_ctr);
    THM_HIP(hipGetLastError());
}
template <class T>
void launch_cgs_update(const Batch &B, const int32_t *mask, const int32_t *jcnt, const T *V, int64_t ld, T *w,
                       double *h, int ldh, bool fused, const double *part, double *npart, int32_t *jcol,
                       int32_t *actc, hipStream_t st) {
    VGUARD(B);
    k_cgs_update<T><<<B.vs.nblocks, 256, sizeof(double) * B.maxcols, st>>>(
        B.off.p, B.len.p, B.vs.blkoff.p, B.ds.blkoff.p, B.ns, mask, jcnt, V, ld, w, h, ldh, fused ? 1 : 0, part,
        B.maxcols, npart, jcol, actc);
    THM_HIP(hipGetLastError());
}
template <class T>
void launch_norm2(const Batch &B, const int32_t *mask, const T *x, double *part, hipStream_t st) {
    VGUARD(B);
    k_norm2<T><<<VGRID(B.vs)>>>(B.off.p, B.len.p, B.vs.blkoff.p, B.ns, mask, x, part);
    THM_HIP(hipGetLastError());
}
template <class TI, class TO>
void launch_scale(const Batch &B, const int32_t *mask, const double *scal, int invert, const TI *x, TO *y1,
                  const int32_t *jcol, int64_t ld1, TO *y2, hipStream_t st) {
    VGUARD(B);
    k_scale<TI, TO><<<VGRID(B.vs)>>>(B.off.p, B.len.p, B.vs.blkoff.p, B.ns, mask, scal, invert, x, y1, jcol, ld1, y2);
    THM_HIP(hipGetLastError());
}
template <class T>
void launch_lincomb(const Batch &B, const int32_t *mask, const int32_t *kcnt, const T *V, int64_t ld,
                    const double *coef, int ldc, T *y, hipStream_t st) {
    VGUARD(B);
    k_lincomb<T><<<VGRID(B.vs)>>>(B.off.p, B.len.p, B.vs.blkoff.p, B.ns, mask, kcnt, V, ld, coef, ldc, y);
    THM_HIP(hipGetLastError());
}
template <class TX, class TZ>
void launch_axpy(const Batch &B, const int32_t *mask, const double *scal, const TZ *z, TX *x, hipStream_t st) {
    VGUARD(B);
    k_axpy<TX, TZ><<<VGRID(B.vs)>>>(B.off.p, B.len.p, B.vs.blkoff.p, B.ns, mask, scal, z, x);
    THM_HIP(hipGetLastError());
}
void launch_norm_finish(const Batch &B, const double *part, const int32_t *mask, double *out, const double *bnorm,
                        double rtol, double *resid, int32_t *running, hipStream_t st) {
    k_norm_finish<<<B.ns, 256, 0, st>>>(B.ns, B.vs.blkoff.p, part, mask, out, bnorm, rtol,
                                                   resid, running);
    THM_HIP(hipGetLastError());
}
void launch_reduce_cols(const Batch &B, const int32_t *mask, const int32_t *jcnt, const double *part, double *out,
                        int ldo, int accumulate, hipStream_t st) {
    k_reduce_cols<<<dim3(B.ns, (B.maxcols + 31) / 32), 256, 0, st>>>(B.ds.blkoff.p, B.ns, mask, jcnt, part,
                                                                      B.maxcols, out, ldo, accumulate);
    THM_HIP(hipGetLastError());
}
void launch_cycle_start(const Batch &B, const double *part, int32_t *running, int32_t *active, int32_t *jcnt,
                        const double *bnorm, const double *rtol_d, double *g, int m, double *beta, double *resid,
                        int32_t *iters, int max_iter, int32_t *step_ctr, int32_t *hrun, hipStream_t st,
                        const double *resid0, int32_t *stepped) {
    k_cycle_start<<<B.ns, 256, 0, st>>>(B.ns, B.vs.blkoff.p, part, running, active, jcnt, bnorm, rtol_d,
                                       g, m, beta, resid, iters, max_iter, step_ctr, hrun, resid0, stepped);
    THM_HIP(hipGetLastError());
}
template <class T>
void launch_arnoldi_close(const Batch &B, const double *npart, const int32_t *jcol, const int32_t *actc, const T *w,
                          T *V, int64_t ld, T *cur, const double *hcol, int ldh, double *H, double *cs, double *sn,
                          double *g, int32_t *active, int32_t *jcnt, double *hnext, const double *bnorm,
                          const double *rtol_d, int m, int32_t *iters, int max_iter, double *est, int32_t *hflags,
                          const int32_t *step_ctr, int spc, int nslots, hipStream_t st) {
    if (m > 1024) fail(THM_EINVAL, "restart must be <= 1024");
    k_arnoldi_close<T><<<B.vs.nblocks + B.ns, 256, 0, st>>>(
        B.off.p, B.len.p, B.vs.blkoff.p, B.vs.nblocks, B.ns, npart, jcol, actc, w, V, ld, cur, hcol, ldh, H, cs, sn, g,
        active, jcnt, hnext, bnorm, rtol_d, m, iters, max_iter, est, hflags, step_ctr, spc, nslots);
    THM_HIP(hipGetLastError());
}
void launch_hsolve(const Batch &B, const int32_t *running, const int32_t *jcnt, const double *H, const double *g,
                   double *y, int m, hipStream_t st) {
    k_hsolve<<<B.ns, 64, 0, st>>>(B.ns, running, jcnt, H, g, y, m);
    THM_HIP(hipGetLastError());
}
template <class T>
void launch_zero_flagged(const Batch &B, const uint8_t *const *dirs, T *x, hipStream_t st) {
    if (!B.es.nblocks) return;
    k_zero_flagged<T><<<B.es.nblocks, 256, 0, st>>>(B.off.p, B.nvec.p, B.es.blkoff.p, B.ns, dirs, x);
    THM_HIP(hipGetLastError());
}

#define INST_T(T)                                                                                             \
    template void launch_dots<T>(const Batch &, const int32_t *, const int32_t *, const T *, int64_t, const T *,   \
                                 double *, int, int32_t *, hipStream_t);                                      \
    template void launch_cgs_update<T>(const Batch &, const int32_t *, const int32_t *, const T *, int64_t, T *,   \
                                       double *, int, bool, const double *, double *, int32_t *, int32_t *,   \
                                       hipStream_t);                                                          \
    template void launch_arnoldi_close<T>(const Batch &, const double *, const int32_t *, const int32_t *,    \
                                          const T *, T *, int64_t, T *, const double *, int, double *, double *,   \
                                          double *, double *, int32_t *, int32_t *, double *, const double *, \
                                          const double *, int, int32_t *, int, double *, int32_t *,           \
                                          const int32_t *, int, int, hipStream_t);                            \
    template void launch_norm2<T>(const Batch &, const int32_t *, const T *, double *, hipStream_t);          \
    template void launch_lincomb<T>(const Batch &, const int32_t *, const int32_t *, const T *, int64_t,      \
                                    const double *, int, T *, hipStream_t);                                   \
    template void launch_zero_flagged<T>(const Batch &, const uint8_t *const *, T *, hipStream_t);
INST_T(double)
INST_T(float)
template void launch_scale<double, double>(const Batch &, const int32_t *, const double *, int, const double *,
                                           double *, const int32_t *, int64_t, double *, hipStream_t);
template void launch_scale<float, float>(const Batch &, const int32_t *, const double *, int, const float *,
                                         float *, const int32_t *, int64_t, float *, hipStream_t);
template void launch_scale<float, double>(const Batch &, const int32_t *, const double *, int, const float *,
                                          double *, const int32_t *, int64_t, double *, hipStream_t);
template void launch_scale<double, float>(const Batch &, const int32_t *, const double *, int, const double *,
                                          float *, const int32_t *, int64_t, float *, hipStream_t);
template void launch_axpy<double, double>(const Batch &, const int32_t *, const double *, const double *, double *,
                                          hipStream_t);
template void launch_axpy<float, float>(const Batch &, const int32_t *, const double *, const float *, float *,
                                        hipStream_t);
template void launch_axpy<double, float>(const Batch &, const int32_t *, const double *, const float *, double *,
                                         hipStream_t);

}  // namespace thm
