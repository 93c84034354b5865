// y = (K +- iC) x and y = b - (K +- iC) x from the cells, without the assembled K.
//
// All cells of a system have the same size, so the matrix of cell c is
//     K_c = curl / mu_c - w^2 eps_c mass
// with two reference matrices per system: two products of a small matrix with the columns x_c of all
// cells, which the matrix cores do.  A wave takes 8 (cell, member) pairs, 16 real columns; members are systems
// with the same K.  Rows of cell-interior functions belong to one cell and go to y; the others go to
// z, and a second launch adds the two to four cells of such a row in their order, applies C from
// its rows and leaves x on Dirichlet rows.
//
// The assembled product is bound by the matrix (12 bytes an entry) or, in groups, by the gathers of
// x through the caches.  Here a cell reads its x once for all its rows, and what is left is x,
// y, z and the cells' indices: 256^2 cells of degree 2, FP64, 87 -> 35 us (25 and 10, 13 at the copy
// rate), FP32 60 -> 28; sixteen members of 64^2 cells, FP64, 54 -> 35.  The two terms have sums of
// their own, scaled at the end: the error stays at or below that of the assembled forms (FP32, the
// same mesh: 6.2e-8 relative against 6.6e-8 to 7.9e-8; factors on x: 7.4e-8).
#include "kernels.h"

namespace thm {

template <class T> struct CellMma;
template <> struct CellMma<float> {
    typedef float v4 __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ v4 op(float a, float b, v4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int g, int v) { return 4 * g + v; }
};
template <> struct CellMma<double> {
    typedef double v4 __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ v4 op(double a, double b, v4 c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int g, int v) { return g + 4 * v; }
};
template <class T> __device__ __forceinline__ const T *cell_frag(const CellDesc &d);
template <> __device__ __forceinline__ const float *cell_frag<float>(const CellDesc &d) { return d.frag32; }
template <> __device__ __forceinline__ const double *cell_frag<double>(const CellDesc &d) { return d.frag64; }

// The reference matrices in the lane order of the products' left operand:
// [curl, mass][row tile][4 columns][lane], zero padded.  ref holds the mass first.
__global__ void __launch_bounds__(256) k_cell_frag(int nl, const double *__restrict__ ref, double *__restrict__ f64,
                                                   float *__restrict__ f32) {
    const int ks = (nl + 3) / 4, mt = (nl + 15) / 16, e = blockIdx.x * 256 + threadIdx.x;
    if (e >= 2 * mt * ks * 64) return;
    const int lane = e & 63, k = 4 * (e / 64 % ks) + (lane >> 4), r = 16 * (e / 64 / ks % mt) + (lane & 15);
    const double v = r < nl && k < nl ? ref[(e / 64 / ks / mt ? 0 : nl * nl) + r * nl + k] : 0.0;
    f64[e] = v;
    f32[e] = (float)v;
}
// DoFs of the cells' functions that are not interior, -1 on Dirichlet sides
__global__ void __launch_bounds__(256) k_cell_index(int64_t ncells, int nl, int ne, const int32_t *__restrict__ dofs,
                                                    const uint8_t *__restrict__ dir, int32_t *__restrict__ idx) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= ncells * ne) return;
    const int32_t q = dofs[e / ne * nl + e % ne];
    idx[e] = dir[q] ? -1 : q;
}

template <class T, int KS>
__device__ __forceinline__ void cell_tile(const CellDesc &d, const SpmvGroup &G, int tile, const T *frag,
                                          const int64_t *__restrict__ off, const int32_t *__restrict__ mask,
                                          const T *__restrict__ xb, T *__restrict__ yb, const T *__restrict__ bb,
                                          T *__restrict__ zb) {
    using V4 = typename CellMma<T>::v4;
    constexpr int MT = (4 * KS + 15) / 16;
    const int lane = threadIdx.x & 63, g = lane >> 4, comp = lane & 1;
    const uint32_t pair = 8u * tile + ((lane & 15) >> 1), npairs = (uint32_t)d.ncells * G.nm;
    const uint32_t pc = min(pair, npairs - 1), c = pc / (uint32_t)G.nm;
    const int s = G.mem[pc - c * G.nm];
    const bool act = pair < npairs && (!mask || mask[s]);
    if (!__any(act)) return;
    const int nl = d.nl, ne = d.ne, ni = nl - ne;
    const int64_t base = off[s];
    const T *x = xb + base + comp;
    const int32_t *idx = d.idx + (int64_t)c * ne;
    const int32_t in0 = d.nskel + (int32_t)c * ni - ne;  // DoF of interior function k, less k
    int32_t q[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        const int k = 4 * ks + g;
        q[ks] = k < ne ? idx[k] : k < nl ? in0 + k : -1;
    }
    T xv[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) xv[ks] = act && q[ks] >= 0 ? x[2 * (int64_t)q[ks]] : (T)0;
    const T a = (T)(1.0 / d.mu[c]), m = (T)(d.eps ? d.w2 * d.eps[c] : d.w2);
    V4 acc[MT], am[MT];
#pragma unroll
    for (int t = 0; t < MT; ++t) acc[t] = am[t] = V4{0, 0, 0, 0};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int t = 0; t < MT; ++t) {
            acc[t] = CellMma<T>::op(frag[(t * KS + ks) * 64 + lane], xv[ks], acc[t]);
            am[t] = CellMma<T>::op(frag[((MT + t) * KS + ks) * 64 + lane], xv[ks], am[t]);
        }
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[t][v] = a * acc[t][v] - m * am[t][v];
    if (!act) return;
    T *z = zb + 2 * (d.zoff + (int64_t)pair * ne) + comp;
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int r = 16 * t + CellMma<T>::row(g, v);
            if (r < ne) {
                z[2 * r] = acc[t][v];
            } else if (r < nl) {
                const int64_t o = base + comp + 2 * (int64_t)(in0 + r);
                yb[o] = bb ? bb[o] - acc[t][v] : acc[t][v];
            }
        }
}

// rounds: tiles of a wave, so that a block's copy of the reference matrices serves several
template <class T>
__global__ void __launch_bounds__(256) k_cell_product(const CellDesc *__restrict__ ds,
                                                      const SpmvGroup *__restrict__ groups,
                                                      const int32_t *__restrict__ blkoff, int ng, int rounds,
                                                      const int64_t *__restrict__ off,
                                                      const int32_t *__restrict__ mask, const T *__restrict__ xb,
                                                      T *__restrict__ yb, const T *__restrict__ bb,
                                                      T *__restrict__ zb) {
    extern __shared__ __align__(16) char cell_lds[];
    T *frag = reinterpret_cast<T *>(cell_lds);
    const int gi = blkoff[ng + 1 + blockIdx.x];
    const CellDesc &d = ds[gi];
    const SpmvGroup &G = groups[gi];
    const int ks = (d.nl + 3) / 4, n = 2 * ((d.nl + 15) / 16) * ks * 64;
    const T *f = cell_frag<T>(d);
    for (int e = threadIdx.x; e < n; e += 256) frag[e] = f[e];
    __syncthreads();
    const int t0 = ((int)blockIdx.x - blkoff[gi]) * 4 * rounds + (threadIdx.x >> 6);
    for (int r = 0; r < rounds; ++r) {
        const int tile = t0 + 4 * r;
        if (tile >= d.tiles) return;
        switch (ks) {
        case 1: cell_tile<T, 1>(d, G, tile, frag, off, mask, xb, yb, bb, zb); break;
        case 3: cell_tile<T, 3>(d, G, tile, frag, off, mask, xb, yb, bb, zb); break;
        case 6: cell_tile<T, 6>(d, G, tile, frag, off, mask, xb, yb, bb, zb); break;
        case 10: cell_tile<T, 10>(d, G, tile, frag, off, mask, xb, yb, bb, zb); break;
        case 14: cell_tile<T, 14>(d, G, tile, frag, off, mask, xb, yb, bb, zb); break;
        }
    }
}

template <class T> struct CellPair;
template <> struct CellPair<float> { using t = float2; };
template <> struct CellPair<double> { using t = double2; };

template <class T>
__global__ void __launch_bounds__(256) k_cell_rows(const CellDesc *__restrict__ ds, const SpmvGroup *__restrict__ groups,
                                                   const int32_t *__restrict__ blkoff, int ng,
                                                   const MatDesc *__restrict__ mats, const int64_t *__restrict__ off,
                                                   const int32_t *__restrict__ mask, const T *__restrict__ xb,
                                                   T *__restrict__ yb, const T *__restrict__ bb, float csign,
                                                   const T *__restrict__ zb) {
    using T2 = typename CellPair<T>::t;
    const int gi = blkoff[ng + 1 + blockIdx.x];
    const CellDesc &d = ds[gi];
    const SpmvGroup &G = groups[gi];
    const uint32_t e = ((uint32_t)blockIdx.x - blkoff[gi]) * 256u + threadIdx.x;
    const uint32_t mi = e / (uint32_t)d.nskel, r = e - mi * d.nskel;
    if (mi >= (uint32_t)G.nm) return;
    const int s = G.mem[mi];
    if (mask && !mask[s]) return;
    const MatDesc &mat = mats[s];
    const T2 *x = reinterpret_cast<const T2 *>(xb + off[s]);
    const T2 *z = reinterpret_cast<const T2 *>(zb) + d.zoff;
    const int32_t p0 = d.d2c_ptr[r], p1 = d.d2c_ptr[r + 1], c0 = mat.crowptr[r], c1 = mat.crowptr[r + 1];
    T2 a{0, 0};
    if (d.dir[r]) {
        a = x[r];
    } else {
        for (int32_t p = p0; p < p1; ++p) {
            const uint32_t src = d.d2c_src[p], c = src / (uint32_t)d.nl, u = src - c * d.nl;
            const T2 v = z[(int64_t)(c * G.nm + mi) * d.ne + u];
            a.x += v.x;
            a.y += v.y;
        }
        const T *cv = reinterpret_cast<const T *>(mat.cval);
        const T sg = (T)csign;
        for (int32_t p = c0; p < c1; ++p) {
            const T c = sg * cv[p];
            const T2 v = x[mat.ccol[p]];
            a.x -= c * v.y;
            a.y += c * v.x;
        }
    }
    if (bb) {
        const T2 b = reinterpret_cast<const T2 *>(bb + off[s])[r];
        a = T2{b.x - a.x, b.y - a.y};
    }
    reinterpret_cast<T2 *>(yb + off[s])[r] = a;
}

void launch_cell_setup(int64_t ncells, int nl, int ne, const double *ref, const int32_t *dofs, const uint8_t *dir,
                       double *frag64, float *frag32, int32_t *idx, hipStream_t st) {
    k_cell_frag<<<(cell_frag_size(nl) + 255) / 256, 256, 0, st>>>(nl, ref, frag64, frag32);
    if (ne > 0) k_cell_index<<<(unsigned)((ncells * ne + 255) / 256), 256, 0, st>>>(ncells, nl, ne, dofs, dir, idx);
    THM_HIP(hipGetLastError());
}

template <class T>
void launch_spmv_cells(const CellBatch &C, const MatDesc *mats, const SpmvGroup *groups, const int64_t *off,
                       const int32_t *mask, const T *x, T *y, const T *b, float csign, hipStream_t st) {
    T *z = reinterpret_cast<T *>(C.z.p);
    const int ng = (int)C.desc.n;
    k_cell_product<T><<<C.tiles.nblocks, 256, sizeof(T) * C.frag_max, st>>>(C.desc.p, groups, C.tiles.blkoff.p, ng,
                                                                           C.rounds, off, mask, x, y, b, z);
    k_cell_rows<T><<<C.rows.nblocks, 256, 0, st>>>(C.desc.p, groups, C.rows.blkoff.p, ng, mats, off, mask, x, y, b,
                                                   csign, z);
    THM_HIP(hipGetLastError());
}
template void launch_spmv_cells<double>(const CellBatch &, const MatDesc *, const SpmvGroup *, const int64_t *,
                                        const int32_t *, const double *, double *, const double *, float, hipStream_t);
template void launch_spmv_cells<float>(const CellBatch &, const MatDesc *, const SpmvGroup *, const int64_t *,
                                       const int32_t *, const float *, float *, const float *, float, hipStream_t);

}  // namespace thm
