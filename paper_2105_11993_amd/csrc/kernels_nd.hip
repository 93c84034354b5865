// Nested-dissection form of K^{-1} (see nd.h): front assembly, small dense inverses and the
// packing of the apply matrices (setup), and the application.
//
// Words per application against the layered forms: a box of w x w cells with (p + 1) DoFs per
// edge is cut by lines of O(w (p + 1)) DoFs, so all boxes of one size keep O(N) words together
// and the whole factor O(N log N), where cyclic reduction over layers of width O(sqrt N) keeps
// O(N^1.5).  Measured, against cyclic reduction (2D) and block LU (3D): one allocation-free
// application on 64^2 cells of degree 2 in FP64 68 instead of 140 us (60 when repeated on the same
// vectors); a GMRES step on 11 x 9 x 10 cells of degree 1 177 instead of 565 us; the first solve there,
// with the factorisation, 110 instead of 504 ms.
#include "nd.h"

namespace thm {

__device__ __forceinline__ int nd_find(const int32_t *blkoff, int n, int b) { return blkoff[n + 1 + b]; }

// ------------------------------------------------------------------ factorisation
// Front of a leaf: the condensed matrices of its cells added one after the other (fixed
// order), Dirichlet rows as the identity.
__global__ void __launch_bounds__(256) k_nd_leaf(const NdFront *__restrict__ fr) {
    const NdFront f = fr[blockIdx.x];
    const int n = f.b + f.c, ne = f.ne;
    for (int64_t e = threadIdx.x; e < (int64_t)n * n; e += 256) {
        const int i = (int)(e / n), j = (int)(e - (int64_t)i * n);
        f.F[e] = (i == j && i < f.b && f.dir[f.own[i]]) ? 1.0 : 0.0;
    }
    for (int q = 0; q < f.ncell; ++q) {
        __syncthreads();
        const double *k = f.kcond + (int64_t)f.cell[q] * ne * ne;
        const int32_t *r = f.row + (int64_t)q * ne;
        for (int e = threadIdx.x; e < ne * ne; e += 256) {
            const int u = e / ne, v = e - u * ne;
            f.F[(int64_t)r[u] * n + r[v]] += k[e];
        }
    }
}

// Front of an upper node: the Schur complements of its children, each entry summed over the
// children that hold both its row and its column, in child order.
__global__ void __launch_bounds__(256) k_nd_merge(const NdFront *__restrict__ fr, const int32_t *__restrict__ blkoff,
                                                  int nf) {
    const int q = nd_find(blkoff, nf, blockIdx.x);
    const NdFront f = fr[q];
    const int n = f.b + f.c, kc = f.kc;
    const int64_t e = (int64_t)(blockIdx.x - blkoff[q]) * 256 + threadIdx.x;
    if (e >= (int64_t)n * n) return;
    const int i = (int)(e / n), j = (int)(e - (int64_t)i * n);
    double a = (i == j && i < f.b && f.dir[f.own[i]]) ? 1.0 : 0.0;
    for (int x = 0; x < kc; ++x) {
        const int ci = f.cnode[(int64_t)i * kc + x];
        if (ci < 0) break;  // lists are filled from the front
        for (int y = 0; y < kc; ++y) {
            const int cj = f.cnode[(int64_t)j * kc + y];
            if (cj != ci) continue;
            const NdChild h = f.child[ci];
            a += h.U[(int64_t)(f.cidx[(int64_t)i * kc + x] - h.uoff) * h.ld + (f.cidx[(int64_t)j * kc + y] - h.uoff)];
            break;
        }
    }
    f.F[e] = a;
}

// Dinv = F_oo^{-1} by Gauss-Jordan with partial pivoting in LDS, one workgroup per front with
// b <= ND_INV_MAX.  Rows stay in place: with p_k the pivot row of column k, the inverse is
// Dinv[k][p_j] = A[p_k][j].  Bound by the LDS traffic of the rank-1 updates.
constexpr int NDI_T = 512;
__global__ void __launch_bounds__(NDI_T) k_nd_invert(const NdFront *__restrict__ fr) {
    extern __shared__ __align__(16) double ndi_lds[];
    __shared__ int piv[ND_INV_MAX], used[ND_INV_MAX];
    __shared__ double prow[ND_INV_MAX], fcol[ND_INV_MAX];
    const NdFront f = fr[blockIdx.x];
    const int n = f.b, nf = f.b + f.c, ld = n | 1;
    if (n == 0 || n > ND_INV_MAX) return;  // the whole block
    double *A = ndi_lds;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int i = wave; i < n; i += NDI_T / 64)
        for (int j = lane; j < n; j += 64) A[i * ld + j] = f.F[(int64_t)i * nf + j];
    if (threadIdx.x < ND_INV_MAX) used[threadIdx.x] = 0;
    __syncthreads();
    for (int k = 0; k < n; ++k) {
        if (wave == 0) {
            double best = -1.0;
            int at = 0x7fffffff;
            for (int r = lane; r < n; r += 64) {
                const double v = used[r] ? -1.0 : fabs(A[r * ld + k]);
                if (v > best) {
                    best = v;
                    at = r;
                }
            }
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) {
                const double v = __shfl_xor(best, o, 64);
                const int w = __shfl_xor(at, o, 64);
                if (v > best || (v == best && w < at)) {
                    best = v;
                    at = w;
                }
            }
            if (lane == 0) {
                if (!(best > 0.0) || !isfinite(best)) {
                    atomicOr(f.status, 1);
                    if (at >= n)  // a column of NaN: any unused row (the status reports it)
                        for (at = 0; used[at];) ++at;
                }
                piv[k] = at;
                used[at] = 1;
            }
        }
        __syncthreads();
        const int p = piv[k];
        const double pv = A[p * ld + k];
        const double ipv = pv != 0.0 ? 1.0 / pv : 0.0;
        for (int t = threadIdx.x; t < 2 * n; t += NDI_T) {
            if (t < n) prow[t] = t == k ? ipv : A[p * ld + t] * ipv;
            else fcol[t - n] = A[(t - n) * ld + k];
        }
        __syncthreads();
        for (int i = wave; i < n; i += NDI_T / 64) {
            const double fi = fcol[i];
            for (int j = lane; j < n; j += 64) {
                double *a = A + i * ld + j;
                if (i == p) *a = prow[j];
                else *a = (j == k ? 0.0 : *a) - fi * prow[j];
            }
        }
        __syncthreads();
    }
    for (int i = wave; i < n; i += NDI_T / 64)
        for (int j = lane; j < n; j += 64) f.Dinv[(int64_t)i * n + piv[j]] = A[piv[i] * ld + j];
}

__global__ void __launch_bounds__(256) k_nd_own(const double *__restrict__ F, int n, int b, double *__restrict__ A) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= (int64_t)b * b) return;
    const int64_t i = e / b;
    A[e] = F[i * n + (e - i * b)];
}

// Slot e of an apply matrix with padded row length ld: tiles of ND_RT rows x 4 P columns (P
// values per 16 bytes), lane l of a wave holding row l % 16 and columns P (l / 16) .. + P of a
// tile, tiles one after another along a row tile.
template <class T>
__device__ __forceinline__ void nd_slot(int64_t e, int ld, int &r, int &c) {
    constexpr int P = 16 / (int)sizeof(T);
    const int64_t rt = e / (ND_RT * (int64_t)ld);
    const int w = (int)(e - rt * ND_RT * ld);
    const int piece = w / (64 * P), l = (w % (64 * P)) / P, t = w % P;
    r = (int)rt * ND_RT + l % 16;
    c = 4 * P * piece + P * (l / 16) + t;
}

__device__ __forceinline__ double nd_value(const NdFront &f, bool fwd, int r, int c) {
    if (fwd) return r < f.c && c < f.b ? f.G[(int64_t)r * f.b + c] : 0.0;
    if (r >= f.b || c >= f.b + f.c) return 0.0;
    return c < f.b ? f.Dinv[(int64_t)r * f.b + c] : -f.G[(int64_t)(c - f.b) * f.b + r];
}

__global__ void __launch_bounds__(256) k_nd_pack(const NdFront *__restrict__ fr, const int32_t *__restrict__ blkoff,
                                                 int nf) {
    const int q = nd_find(blkoff, nf, blockIdx.x);
    const NdFront f = fr[q];
    const int lf = (f.b + ND_KS - 1) / ND_KS * ND_KS, lb = (f.b + f.c + ND_KS - 1) / ND_KS * ND_KS;
    const int64_t nfw = (int64_t)((f.c + ND_RT - 1) / ND_RT * ND_RT) * lf;
    const int64_t nbw = (int64_t)((f.b + ND_RT - 1) / ND_RT * ND_RT) * lb;
    int64_t e = (int64_t)(blockIdx.x - blkoff[q]) * 256 + threadIdx.x;
    if (e >= nfw + nbw) return;
    const bool fwd = e < nfw;
    if (!fwd) e -= nfw;
    const int64_t at = (fwd ? f.fo : f.bo) + e;
    const int ld = fwd ? lf : lb;
    int r, c;
    nd_slot<double>(e, ld, r, c);
    f.m64[at] = nd_value(f, fwd, r, c);
    nd_slot<float>(e, ld, r, c);
    f.m32[at] = (float)nd_value(f, fwd, r, c);
}

constexpr double ND_GROWTH_MIN = ND_GROWTH[0];
// Largest |G| beyond ND_GROWTH[0] (as bits: non-negative doubles order as integers); infinity where an
// entry is not a number.
__global__ void __launch_bounds__(256) k_nd_growth(const NdFront *__restrict__ fr) {
    const NdFront f = fr[blockIdx.x];
    double v = 0.0;
    for (int64_t e = threadIdx.x; e < (int64_t)f.b * f.c; e += 256) {
        const double g = fabs(f.G[e]);
        v = g <= HUGE_VAL ? fmax(v, g) : HUGE_VAL;
    }
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    if ((threadIdx.x & 63) == 0 && v > ND_GROWTH_MIN) atomicMax(f.growth, __double_as_longlong(v));
}

void launch_nd_growth(const std::vector<NdFront> &h, const NdFront *d, hipStream_t st) {
    if (h.empty()) return;
    k_nd_growth<<<(unsigned)h.size(), 256, 0, st>>>(d);
    THM_HIP(hipGetLastError());
}

void launch_nd_leaf(const std::vector<NdFront> &h, const NdFront *d, hipStream_t st) {
    if (h.empty()) return;
    k_nd_leaf<<<(unsigned)h.size(), 256, 0, st>>>(d);
    THM_HIP(hipGetLastError());
}

void launch_nd_merge(const std::vector<NdFront> &h, const NdFront *d, hipStream_t st) {
    std::vector<int64_t> u(h.size());
    for (size_t i = 0; i < h.size(); ++i) u[i] = (int64_t)(h[i].b + h[i].c) * (h[i].b + h[i].c);
    Sched sc;
    sc.build(u, 256, st);
    if (sc.nblocks) k_nd_merge<<<sc.nblocks, 256, 0, st>>>(d, sc.blkoff.p, (int)h.size());
    THM_HIP(hipGetLastError());
    THM_HIP(hipStreamSynchronize(st));  // the schedule ends here
}

void launch_nd_invert(const std::vector<NdFront> &h, const NdFront *d, hipStream_t st) {
    int n = 0;
    for (const NdFront &f : h)
        if (f.b <= ND_INV_MAX) n = std::max(n, f.b);
    if (!n) return;
    const size_t lds = sizeof(double) * n * (n | 1);
    // per device, so before every launch; a refusal shows there
    (void)hipFuncSetAttribute(reinterpret_cast<const void *>(k_nd_invert), hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)(sizeof(double) * ND_INV_MAX * (ND_INV_MAX | 1)));
    k_nd_invert<<<(unsigned)h.size(), NDI_T, lds, st>>>(d);
    THM_HIP(hipGetLastError());
}

void launch_nd_own(const double *F, int n, int b, double *A, hipStream_t st) {
    if (!b) return;
    k_nd_own<<<(unsigned)(((int64_t)b * b + 255) / 256), 256, 0, st>>>(F, n, b, A);
    THM_HIP(hipGetLastError());
}

void launch_nd_pack(const std::vector<NdFront> &h, const NdFront *d, hipStream_t st) {
    std::vector<int64_t> u(h.size());
    for (size_t i = 0; i < h.size(); ++i)
        u[i] = nd_pad(h[i].c, ND_RT) * nd_pad(h[i].b, ND_KS) + nd_pad(h[i].b, ND_RT) * nd_pad(h[i].b + h[i].c, ND_KS);
    Sched sc;
    sc.build(u, 256, st);
    if (sc.nblocks) k_nd_pack<<<sc.nblocks, 256, 0, st>>>(d, sc.blkoff.p, (int)h.size());
    THM_HIP(hipGetLastError());
    THM_HIP(hipStreamSynchronize(st));  // the schedule ends here
}

// ------------------------------------------------------------------ application
// A block serves some row tiles of one node and direction, Y = M X with
//   up:    M = G (c x b),                   X = r,               u = (children's u) + Y
//   down:  M = [Dinv | -G^T] (b x (b + c)), X = [r; x_boundary], x = Y,
// where r = rhs - (children's u on the own DoFs) is formed while X is read (both directions form
// it, so no phase writes what another block of it reads).  A block has four or eight waves; ks of
// them share one 16-row tile and split its columns, the others take the next
// tiles.  A wave streams its tiles as contiguous 1 KiB runs (nd_slot), the first of them
// requested before X is staged.  Vectors are position-major, the (re, im) pairs of a factor
// group's members side by side.  The sums have a fixed order.
//
// What bounds it: the chain of dependent reads of a phase (block descriptor, index lists,
// vectors) for small trees, the matrices' bytes for large ones.  The index lists of a thread's
// staged entries are therefore read together, without branches (absent children read entry 0
// and are dropped by a select).
template <class T>
struct NdVec {
    typedef T vec __attribute__((ext_vector_type(16 / sizeof(T))));
    static constexpr int P = 16 / (int)sizeof(T);
};
template <class T> struct NdPair;
template <> struct NdPair<double> { using t = double2; };
template <> struct NdPair<float> { using t = float2; };

// Workgroups are dealt to the 8 XCDs round-robin; renumber them so that the row tiles of one
// node, which read the same vectors, run on one XCD.
__device__ __forceinline__ int nd_block() {
    const int nb = gridDim.x, b = blockIdx.x;
    const int q = nb >> 3, rem = nb & 7, x = b & 7, i = b >> 3;
    return x < rem ? x * (q + 1) + i : rem * (q + 1) + (x - rem) * q + i;
}

constexpr int ND_UNR = 4;  // tiles in flight per wave

// Columns [k0, k0 + kn) of X for the block's member, handed to put(k, value).  KC: children lists
// per own row.
template <class T, bool FWD, int KC, class Put>
__device__ __forceinline__ void nd_stage_kc(const NdTask &tk, int k0, int kn, int K, const typename NdPair<T>::t *ws,
                                            const typename NdPair<T>::t *ys, const typename NdPair<T>::t *ub, Put put) {
    using T2 = typename NdPair<T>::t;
    constexpr int U = 2;
    const int nt = blockDim.x;
    for (int s0 = threadIdx.x; s0 < kn; s0 += nt * U) {
        int j[U], ch[U][KC ? KC : 1];
        bool own[U], ok[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int s = s0 + nt * u, kk = k0 + s;
            ok[u] = s < kn && kk < K;
            own[u] = FWD || !ok[u] || kk < tk.b;
            j[u] = own[u] ? (ok[u] ? kk : 0) : tk.bpos[kk - tk.b];
#pragma unroll
            for (int x = 0; x < KC; ++x) ch[u][x] = (ok[u] && own[u]) ? tk.cidx[kk * KC + x] : -1;
        }
        T2 v[U], c[U][KC ? KC : 1];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            v[u] = (own[u] ? ws : ys)[j[u]];
#pragma unroll
            for (int x = 0; x < KC; ++x) c[u][x] = ub[max(ch[u][x], 0)];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int x = 0; x < KC; ++x) {
                v[u].x -= ch[u][x] >= 0 ? c[u][x].x : (T)0;
                v[u].y -= ch[u][x] >= 0 ? c[u][x].y : (T)0;
            }
            if (s0 + nt * u < kn) put(s0 + nt * u, ok[u] ? v[u] : T2{0, 0});
        }
    }
}

template <class T, bool FWD, class Put>
__device__ __forceinline__ void nd_stage(const NdTask &tk, int k0, int kn, int K, const typename NdPair<T>::t *ws,
                                         const typename NdPair<T>::t *ys, const typename NdPair<T>::t *ub, Put put) {
    if (tk.kc == 0) nd_stage_kc<T, FWD, 0>(tk, k0, kn, K, ws, ys, ub, put);
    else if (tk.kc == 1) nd_stage_kc<T, FWD, 1>(tk, k0, kn, K, ws, ys, ub, put);
    else if (tk.kc == 2) nd_stage_kc<T, FWD, 2>(tk, k0, kn, K, ws, ys, ub, put);
    else nd_stage_kc<T, FWD, 4>(tk, k0, kn, K, ws, ys, ub, put);
}

// The children's update of boundary row `row` of a node (member m).
template <class T>
__device__ __forceinline__ typename NdPair<T>::t nd_children(const NdTask &tk, int row, int m,
                                                             const typename NdPair<T>::t *ub) {
    using T2 = typename NdPair<T>::t;
    const int32_t *l = tk.cidx + (int64_t)(tk.b + row) * tk.kc;
    T2 a{0, 0};
    for (int x = 0; x < tk.kc; ++x) {
        const int q = l[x];
        const T2 v = ub[(int64_t)max(q, 0) * (tk.cs / 2) + m];
        a.x += q >= 0 ? v.x : (T)0;
        a.y += q >= 0 ? v.y : (T)0;
    }
    return a;
}

// One member (re, im): the 2-column product on the vector units (the matrix units would idle
// in 14 of 16 columns and have the same FP64 rate).
template <class T, bool FWD>
__global__ void __launch_bounds__(512) k_nd_vec(const NdTask *__restrict__ tasks, const int32_t *__restrict__ memb,
                                                const int32_t *__restrict__ mask, const T *__restrict__ wsb,
                                                T *__restrict__ ysb, T *__restrict__ ubb) {
    using T2 = typename NdPair<T>::t;
    using V = typename NdVec<T>::vec;
    constexpr int P = NdVec<T>::P;
    extern __shared__ __align__(32) char nd_lds[];
    __shared__ T2 part_sum[8][16];
    T2 *xs = reinterpret_cast<T2 *>(nd_lds);
    const NdTask tk = tasks[nd_block()];
    if (mask && !mask[memb[tk.mbeg]]) return;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, i16 = lane & 15, g = lane >> 4;
    const int rows = FWD ? tk.c : tk.b, K = FWD ? tk.b : tk.b + tk.c;
    const int Kp = (K + ND_KS - 1) / ND_KS * ND_KS;
    const int part = wave % tk.ks, nw = blockDim.x >> 6;
    const T2 *ws = reinterpret_cast<const T2 *>(wsb + tk.gbase) + tk.pos0;
    T2 *ys = reinterpret_cast<T2 *>(ysb + tk.gbase);
    T2 *ub = reinterpret_cast<T2 *>(ubb + tk.ubase);
    for (int t0 = 0; t0 < tk.tiles; t0 += nw / tk.ks) {
        const int rt = tk.rt0 + t0 + wave / tk.ks, row = rt * ND_RT + i16;
        const bool live = t0 + wave / tk.ks < tk.tiles && rt * ND_RT < rows;
        const bool out = live && part == 0 && g == 0 && row < rows;
        const V *M = reinterpret_cast<const V *>(static_cast<const T *>(tk.M) + (int64_t)(live ? rt : 0) * ND_RT * Kp) +
                     lane;
        T ar = 0, ai = 0;
        T2 add{0, 0};
        for (int k0 = 0; k0 < max(Kp, 1); k0 += ND_KC_VEC) {
            const int kn = min(ND_KC_VEC, Kp - k0);
            const int np = kn / (4 * P), per = (np + tk.ks - 1) / tk.ks;
            const int pb = part * per, pe = live ? min(np, pb + per) : pb;
            const V *Mc = M + (int64_t)(k0 / (4 * P)) * 64;
            V cur[ND_UNR];
            if (pb < pe) {
#pragma unroll
                for (int u = 0; u < ND_UNR; ++u) cur[u] = Mc[(int64_t)min(pb + u, pe - 1) * 64];
            }
            if (t0 == 0 || Kp > ND_KC_VEC) {
                if (t0 || k0) __syncthreads();
                nd_stage<T, FWD>(tk, k0, kn, K, ws, ys, ub, [&](int k, T2 v) { xs[k] = v; });
                __syncthreads();
            }
            if (FWD && k0 == 0 && out) add = nd_children<T>(tk, row, 0, ub);
            for (int q = pb; q < pe; q += ND_UNR) {
                V nxt[ND_UNR];
#pragma unroll
                for (int u = 0; u < ND_UNR; ++u) nxt[u] = Mc[(int64_t)min(q + ND_UNR + u, pe - 1) * 64];
#pragma unroll
                for (int u = 0; u < ND_UNR; ++u) {
                    if (q + u >= pe) break;
                    const T2 *x = xs + 4 * P * (q + u) + P * g;
#pragma unroll
                    for (int t = 0; t < P; ++t) {
                        const T2 v = x[t];
                        ar += cur[u][t] * v.x;
                        ai += cur[u][t] * v.y;
                    }
                }
#pragma unroll
                for (int u = 0; u < ND_UNR; ++u) cur[u] = nxt[u];
            }
        }
        // sum over the four lane groups, then over the waves that share the tile
#pragma unroll
        for (int o = 16; o < 64; o <<= 1) {
            ar += __shfl_xor(ar, o, 64);
            ai += __shfl_xor(ai, o, 64);
        }
        if (tk.ks > 1) {
            if (t0) __syncthreads();
            if (g == 0) part_sum[wave][i16] = T2{ar, ai};
            __syncthreads();
            if (out)
                for (int w = 1; w < tk.ks; ++w) {
                    const T2 v = part_sum[wave + w][i16];
                    ar += v.x;
                    ai += v.y;
                }
        }
        if (!out) continue;
        if (FWD) ub[tk.uoff + row] = T2{add.x + ar, add.y + ai};
        else ys[tk.pos0 + row] = T2{ar, ai};
    }
}

// Matrix-core form for groups of members: NNT tiles of 8 members (16 columns) per block.
template <class T> struct NdMma;
template <> struct NdMma<float> {
    typedef float v4 __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ v4 op(float a, float b, v4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int g, int v) { return 4 * g + v; }
};
template <> struct NdMma<double> {
    typedef double v4 __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ v4 op(double a, double b, v4 c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int g, int v) { return g + 4 * v; }
};

// Every wave reads its part of X straight into the operand registers: a position holds the members'
// (re, im) pairs side by side, so 16 columns of 4 positions are four contiguous runs, and a wave is
// the only reader of its columns in a block of ks = 4.  Staged in LDS instead, a block waited
// for the lists and vectors of all its columns before its first product, in one to five rounds with
// two barriers each, and held 64 KiB: 64^2 cells of degree 2, sixteen members, FP64, the phase
// of 288 + 192 columns 98 -> 52 us; 32^2 cells, FP32, the root of 576 columns 17.5 -> 8.9 us.
// Columns of absent members read the last member's: they only reach outputs that are not stored.
template <class T, bool FWD, int KC, int NNT>
__device__ __forceinline__ void nd_mfma_tile(const NdTask &tk, typename NdMma<T>::v4 (&acc)[NNT],
                                             const typename NdVec<T>::vec *M, int pb, int pe, int K,
                                             const T *__restrict__ ws, const T *__restrict__ ys,
                                             const T *__restrict__ ub) {
    using V = typename NdVec<T>::vec;
    constexpr int P = NdVec<T>::P, U = 8 / P;  // 8 positions of a lane in flight
    const int lane = threadIdx.x & 63, i16 = lane & 15, g = lane >> 4;
    const int b = tk.b;
    const int64_t cs = tk.cs;
    int col[NNT];
#pragma unroll
    for (int nt = 0; nt < NNT; ++nt) col[nt] = min(16 * nt + i16, 2 * tk.nm - 1);
    for (int q = pb; q < pe; q += U) {
        V a[U];
#pragma unroll
        for (int u = 0; u < U; ++u) a[u] = M[(int64_t)min(q + u, pe - 1) * 64];
        T x[U][P][NNT];
        const int k0 = 4 * P * q;
        if (!FWD && k0 >= b && K > b) {  // boundary positions only: the same in the whole wave
            int pos[U][P];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int t = 0; t < P; ++t) pos[u][t] = tk.bpos[min(k0 + 4 * P * u + P * g + t, K - 1) - b];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int t = 0; t < P; ++t)
#pragma unroll
                    for (int nt = 0; nt < NNT; ++nt) x[u][t][nt] = ys[pos[u][t] * cs + col[nt]];
        } else {
            int pos[U][P], ch[U][P][KC ? KC : 1];
            bool own[U][P];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int t = 0; t < P; ++t) {
                    const int k = min(k0 + 4 * P * u + P * g + t, K - 1);
                    own[u][t] = FWD || k < b;
                    pos[u][t] = own[u][t] ? k : tk.bpos[k - b];
#pragma unroll
                    for (int c = 0; c < KC; ++c) ch[u][t][c] = own[u][t] ? tk.cidx[k * KC + c] : -1;
                }
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int t = 0; t < P; ++t)
#pragma unroll
                    for (int nt = 0; nt < NNT; ++nt) {
                        T v = (own[u][t] ? ws : ys)[pos[u][t] * cs + col[nt]];
                        T w[KC ? KC : 1];
#pragma unroll
                        for (int c = 0; c < KC; ++c) w[c] = ub[max(ch[u][t][c], 0) * cs + col[nt]];
#pragma unroll
                        for (int c = 0; c < KC; ++c) v -= ch[u][t][c] >= 0 ? w[c] : (T)0;
                        x[u][t][nt] = v;
                    }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (q + u >= pe) break;
#pragma unroll
            for (int t = 0; t < P; ++t) {
                const bool in = k0 + 4 * P * u + P * g + t < K;  // M is zero there, X need not be finite
#pragma unroll
                for (int nt = 0; nt < NNT; ++nt) acc[nt] = NdMma<T>::op(a[u][t], in ? x[u][t][nt] : (T)0, acc[nt]);
            }
        }
    }
}

template <class T, bool FWD, int NNT>
__device__ __forceinline__ void nd_mfma_tiles(const NdTask &tk, T *lds, const int32_t *__restrict__ memb,
                                              const int32_t *__restrict__ mask, const T *__restrict__ wsb,
                                              T *__restrict__ ysb, T *__restrict__ ubb) {
    using T2 = typename NdPair<T>::t;
    using V = typename NdVec<T>::vec;
    using V4 = typename NdMma<T>::v4;
    constexpr int P = NdVec<T>::P;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, i16 = lane & 15, g = lane >> 4;
    const int rows = FWD ? tk.c : tk.b, K = FWD ? tk.b : tk.b + tk.c;
    const int Kp = (K + ND_KS - 1) / ND_KS * ND_KS;
    const int part = wave % tk.ks, nw = blockDim.x >> 6;
    const int64_t cs = tk.cs;
    const T *ws = wsb + tk.gbase + tk.pos0 * cs + 2 * tk.m0;
    T *ys = ysb + tk.gbase + 2 * tk.m0;
    T *ub = ubb + tk.ubase + 2 * tk.m0;
    const int np = Kp / (4 * P), per = (np + tk.ks - 1) / tk.ks;
    for (int t0 = 0; t0 < tk.tiles; t0 += nw / tk.ks) {
        const int rt = tk.rt0 + t0 + wave / tk.ks;
        const bool live = t0 + wave / tk.ks < tk.tiles && rt * ND_RT < rows;
        const V *M = reinterpret_cast<const V *>(static_cast<const T *>(tk.M) + (int64_t)(live ? rt : 0) * ND_RT * Kp) +
                     lane;
        const int pb = part * per, pe = live ? min(np, pb + per) : pb;
        V4 acc[NNT];
#pragma unroll
        for (int nt = 0; nt < NNT; ++nt) acc[nt] = V4{0, 0, 0, 0};
        if (tk.kc == 0) nd_mfma_tile<T, FWD, 0, NNT>(tk, acc, M, pb, pe, K, ws, ys, ub);
        else if (tk.kc == 1) nd_mfma_tile<T, FWD, 1, NNT>(tk, acc, M, pb, pe, K, ws, ys, ub);
        else if (tk.kc == 2) nd_mfma_tile<T, FWD, 2, NNT>(tk, acc, M, pb, pe, K, ws, ys, ub);
        else nd_mfma_tile<T, FWD, 4, NNT>(tk, acc, M, pb, pe, K, ws, ys, ub);
        // waves sharing a tile: partial tiles through LDS, summed by the first
        if (tk.ks > 1) {
            V4 *red = reinterpret_cast<V4 *>(lds);
            if (t0) __syncthreads();
            if (part > 0)
#pragma unroll
                for (int nt = 0; nt < NNT; ++nt) red[(wave * NNT + nt) * 64 + lane] = acc[nt];
            __syncthreads();
            if (part == 0)
                for (int w = 1; w < tk.ks; ++w)
#pragma unroll
                    for (int nt = 0; nt < NNT; ++nt) {
                        const V4 v = red[((wave + w) * NNT + nt) * 64 + lane];
#pragma unroll
                        for (int t = 0; t < 4; ++t) acc[nt][t] += v[t];
                    }
        }
        if (!live || part != 0) continue;
#pragma unroll
        for (int nt = 0; nt < NNT; ++nt) {
            const int n = 16 * nt + i16;
            if (n >= 2 * tk.nm || (mask && !mask[memb[tk.mbeg + tk.m0 + n / 2]])) continue;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = rt * ND_RT + NdMma<T>::row(g, v);
                if (row >= rows) continue;
                if (FWD) {
                    const T2 c = nd_children<T>(tk, row, n / 2, reinterpret_cast<const T2 *>(ub));
                    ub[(tk.uoff + row) * cs + n] = ((n & 1) ? c.y : c.x) + acc[nt][v];
                } else {
                    ys[(tk.pos0 + row) * cs + n] = acc[nt][v];
                }
            }
        }
    }
}

template <class T, bool FWD>
__global__ void __launch_bounds__(512) k_nd_mfma(const NdTask *__restrict__ tasks, const int32_t *__restrict__ memb,
                                                 const int32_t *__restrict__ mask, const T *__restrict__ wsb,
                                                 T *__restrict__ ysb, T *__restrict__ ubb) {
    extern __shared__ __align__(32) char nd_lds[];
    T *lds = reinterpret_cast<T *>(nd_lds);
    const NdTask tk = tasks[nd_block()];
    if (mask) {
        const int lane = threadIdx.x & 63;
        const bool on = lane < tk.nm && mask[memb[tk.mbeg + tk.m0 + lane]];
        if (!__ballot(on)) return;  // the same in every wave
    }
    if (tk.nm <= 8) nd_mfma_tiles<T, FWD, 1>(tk, lds, memb, mask, wsb, ysb, ubb);
    else nd_mfma_tiles<T, FWD, 2>(tk, lds, memb, mask, wsb, ysb, ubb);
}

template <class T, bool FWD>
static void launch_nd(const NdLaunch &L, const int32_t *memb, const int32_t *mask, const T *ws, T *ys, T *ub,
                      hipStream_t st) {
    const NdTask *t = L.tasks.p;
    if (!L.nblocks) return;
    const size_t lds = L.lds;
    if (L.vec) {
        k_nd_vec<T, FWD><<<L.nblocks, 64 * L.waves, lds, st>>>(t, memb, mask, ws, ys, ub);
    } else {
        k_nd_mfma<T, FWD><<<L.nblocks, 64 * L.waves, lds, st>>>(t, memb, mask, ws, ys, ub);
    }
}

template <class T>
void launch_nd_phases(const std::vector<NdLaunch> &L, const int32_t *memb, const int32_t *mask, const T *ws, T *ys,
                      T *ub, hipStream_t st) {
    for (const NdLaunch &l : L) {
        if (l.fwd) launch_nd<T, true>(l, memb, mask, ws, ys, ub, st);
        else launch_nd<T, false>(l, memb, mask, ws, ys, ub, st);
    }
    THM_HIP(hipGetLastError());
}
template void launch_nd_phases<double>(const std::vector<NdLaunch> &, const int32_t *, const int32_t *, const double *,
                                       double *, double *, hipStream_t);
template void launch_nd_phases<float>(const std::vector<NdLaunch> &, const int32_t *, const int32_t *, const float *,
                                      float *, float *, hipStream_t);

}  // namespace thm
