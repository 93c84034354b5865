// Setup of the block preconditioner diag(K, K)^{-1} (eq. (11)) as an exact
// factorised K^{-1}: static condensation of cell interiors, then nested dissection of the
// skeleton DoFs (setup_nd, nd.h).  THM_FACTOR_FORM selects one of the layered forms instead:
// block cyclic reduction over the layers of skeleton DoFs, or block LU (plan_lu).  The paper approximates K^{-1} by an AMG with direct level transitions;
// here the inverse is exact, so GMRES sees the preconditioned operator
// I + [[0, -K^{-1}C], [K^{-1}C, 0]].
//
// Cyclic reduction on the block-tridiagonal skeleton matrix (diagonal blocks D_i,
// couplings Lo_i between position i and i-1): at every level the odd positions p
// are eliminated with explicit inverses Dinv_p; each even position q keeps
//   Gm_q = Lo_q Dinv_{q-1},  Gp_q = Lo_{q+1}^T Dinv_{q+1},
//   D_q <- D_q - Gm_q Lo_q^T - Gp_q Lo_{q+1},  Lo_q <- -Gm_q Lo_{q-1}.
// Application: reduce the right-hand side upwards (r_q -= Gm_q r_{q-1} + Gp_q r_{q+1}),
// solve the last block, then substitute downwards
// (x_p = Dinv_p r_p - Gp_{p-1}^T x_{p-1} - Gm_{p+1}^T x_{p+1}).
// Systems whose Dirichlet-modified K and element matrices are bitwise identical
// share one factor.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

#include "solver.h"

namespace thm {

static bool same_topology(const thm_system &a, const thm_system &b) {
    const Topo &x = a.topo, &y = b.topo;
    if (x.dim != y.dim || x.p != y.p) return false;
    for (int i = 0; i < 3; ++i)
        if (x.n[i] != y.n[i] || x.h[i] != y.h[i]) return false;
    return a.K.col.size() == b.K.col.size() && a.dir == b.dir;
}

static bool same_values(thm_system &a, thm_system &b, hipStream_t st) {
    DBuf<int32_t> flag(1);
    THM_HIP(hipMemsetAsync(flag.p, 0, sizeof(int32_t), st));
    launch_compare(a.kval.p, b.kval.p, (int64_t)a.K.col.size(), flag.p, st);
    launch_compare(a.kel.p, b.kel.p, (int64_t)a.kel.n, flag.p, st);
    int32_t h = 1;
    THM_HIP(hipMemcpyAsync(&h, flag.p, sizeof(int32_t), hipMemcpyDeviceToHost, st));
    THM_HIP(hipStreamSynchronize(st));
    return h == 0;
}

bool same_matrices(thm_system &a, thm_system &b, hipStream_t st) {
    return same_topology(a, b) && a.K.rowptr == b.K.rowptr && a.K.col == b.K.col && same_values(a, b, st);
}

namespace {
// Work of one factor during setup.
struct Work {
    thm_system *rep;
    Factor *f;
    DBuf<double> D, Lo0;                  // initial diagonal / coupling blocks (layering offsets)
    std::map<int, DBuf<double>> lo;       // per layer: current coupling to the previous position (level > 0)
    std::vector<int> pos;
    const double *lo_ptr(int layer) const {
        auto it = lo.find(layer);
        if (it != lo.end()) return it->second.p;
        return Lo0.p + rep->L.lf_off[layer];
    }
    double *d_ptr(int layer) { return D.p + rep->L.sinv_off[layer]; }
};
}  // namespace

// Padded copies for the apply: each input segment starts at its layer's aligned width,
// the row length is padded to a multiple of the MFMA column step and the row count to a
// multiple of the row tile; stored tile by tile (see k_repack).
static void pad_blocks(Factor &f) {
    int64_t poff = 0;
    auto pad = [&](Factor::Blk &b) {
        int c = 0;
        for (int q = 0; q < b.nseg; ++q) {
            b.seg_pstart[q] = c;
            const int k = b.seg_layer[q];
            c += (int)(f.pboff[k + 1] - f.pboff[k]);
        }
        b.seg_pstart[b.nseg] = c;
        b.ld = (c + BCR_KS - 1) / BCR_KS * BCR_KS;
        if (b.ld > 8 * BCR_TAB)
            fail(THM_EUNSUPPORTED, "a factor block has more columns than the apply kernel supports");
        b.poff = poff;
        poff += (int64_t)(b.rows + BCR_RT - 1) / BCR_RT * BCR_RT * b.ld;
    };
    for (auto &lev : f.fwd)
        for (auto &b : lev) pad(b);
    for (auto &lev : f.bwd)
        for (auto &b : lev) pad(b);
    for (auto &b : f.tops) pad(b);
    f.matp_elems = poff;
}

// Plan the level structure of one factor and the offsets of its apply matrices.
static void plan(Factor &f) {
    const int nL = f.nlayers;
    std::vector<int> pos(nL);
    for (int k = 0; k < nL; ++k) pos[k] = k;
    int64_t off = 0;
    auto blk = [&](int layer, int cols) {
        Factor::Blk b{};
        b.layer = layer;
        b.rows = f.bsize[layer];
        b.cols = cols;
        b.off = off;
        off += (int64_t)b.rows * cols;
        return b;
    };
    f.fwd.clear();
    f.bwd.clear();
    f.fw_at.clear();
    f.bk_at.clear();
    f.level_pos.clear();
    auto total = [&](const std::vector<int> &v) {
        int64_t t = 0;
        for (int k : v) t += f.bsize[k];
        return t;
    };
    constexpr int TOP_BLOCKS = 9;
    constexpr int64_t TOP_ROWS = 6144;
    while (pos.size() > 1 && !((int)pos.size() <= TOP_BLOCKS && total(pos) <= TOP_ROWS)) {
        const int m = (int)pos.size();
        std::vector<Factor::Blk> fw, bk;
        std::map<int, int> fwi, bki;
        for (int i = 1; i < m; i += 2) {
            const int b = f.bsize[pos[i]];
            const int bl = f.bsize[pos[i - 1]];
            const int br = i + 1 < m ? f.bsize[pos[i + 1]] : 0;
            Factor::Blk x = blk(pos[i], b + bl + br);
            x.nseg = 0;
            x.seg_layer[x.nseg] = pos[i]; x.seg_src[x.nseg++] = 0;
            x.seg_layer[x.nseg] = pos[i - 1]; x.seg_src[x.nseg++] = 1;
            if (i + 1 < m) { x.seg_layer[x.nseg] = pos[i + 1]; x.seg_src[x.nseg++] = 1; }
            x.out_dst = 1;
            x.subtract = 0;
            bki[i] = (int)bk.size();
            bk.push_back(x);
        }
        for (int i = 0; i < m; i += 2) {
            const int bl = i > 0 ? f.bsize[pos[i - 1]] : 0;
            const int br = i + 1 < m ? f.bsize[pos[i + 1]] : 0;
            Factor::Blk x = blk(pos[i], bl + br);
            x.nseg = 0;
            if (i > 0) { x.seg_layer[x.nseg] = pos[i - 1]; x.seg_src[x.nseg++] = 0; }
            if (i + 1 < m) { x.seg_layer[x.nseg] = pos[i + 1]; x.seg_src[x.nseg++] = 0; }
            x.out_dst = 0;
            x.subtract = 1;
            fwi[i] = (int)fw.size();
            fw.push_back(x);
        }
        f.fwd.push_back(fw);
        f.bwd.push_back(bk);
        f.fw_at.push_back(fwi);
        f.bk_at.push_back(bki);
        f.level_pos.push_back(pos);
        std::vector<int> even;
        for (int i = 0; i < m; i += 2) even.push_back(pos[i]);
        pos = even;
    }
    // dense inverse of the remaining block-tridiagonal system, one task per block row
    f.top_pos = pos;
    f.top_n = (int)total(pos);
    f.top_off = off;
    f.tops.clear();
    int64_t roff = 0;
    for (int k : pos) {
        Factor::Blk b{};
        b.layer = k;
        b.rows = f.bsize[k];
        b.cols = f.top_n;
        b.off = f.top_off + roff * f.top_n;
        b.nseg = (int)pos.size();
        for (size_t q = 0; q < pos.size(); ++q) {
            b.seg_layer[q] = pos[q];
            b.seg_src[q] = 0;
        }
        b.out_dst = 1;
        b.subtract = 0;
        f.tops.push_back(b);
        roff += f.bsize[k];
    }
    off += (int64_t)f.top_n * f.top_n;
    f.mat_elems = off;
    pad_blocks(f);
}

// Plan of the block-LU form (thick layers): forward task i computes
//   y_i = S_i^{-1} r_i - (S_i^{-1} Lo_i) y_{i-1}        (matrix [S_i^{-1} | -S_i^{-1} Lo_i]),
// backward task i (from the last but one layer down) computes
//   x_i = y_i - (S_i^{-1} Lo_{i+1}^T) x_{i+1}          (subtracting task),
// with the block pivots S_0 = D_0, S_i = D_i - Lo_i S_{i-1}^{-1} Lo_i^T.  One forward and one
// backward level per layer, one task each; no dense last system.
static void plan_lu(Factor &f) {
    const int nL = f.nlayers;
    int64_t off = 0;
    f.fwd.clear();
    f.bwd.clear();
    f.fw_at.clear();
    f.bk_at.clear();
    f.level_pos.clear();
    f.tops.clear();
    f.top_pos.clear();
    f.top_n = 0;
    for (int i = 0; i < nL; ++i) {
        Factor::Blk b{};
        b.layer = i;
        b.rows = f.bsize[i];
        b.cols = f.bsize[i] + (i > 0 ? f.bsize[i - 1] : 0);
        b.off = off;
        off += (int64_t)b.rows * b.cols;
        b.nseg = 0;
        b.seg_layer[b.nseg] = i; b.seg_src[b.nseg++] = 0;
        if (i > 0) { b.seg_layer[b.nseg] = i - 1; b.seg_src[b.nseg++] = 1; }
        b.out_dst = 1;
        b.subtract = 0;
        f.fwd.push_back({b});
    }
    for (int i = 0; i + 1 < nL; ++i) {
        Factor::Blk b{};
        b.layer = i;
        b.rows = f.bsize[i];
        b.cols = f.bsize[i + 1];
        b.off = off;
        off += (int64_t)b.rows * b.cols;
        b.nseg = 0;
        b.seg_layer[b.nseg] = i + 1; b.seg_src[b.nseg++] = 1;
        b.out_dst = 1;
        b.subtract = 1;
        f.bwd.push_back({b});
    }
    f.top_off = off;
    f.mat_elems = off;
    pad_blocks(f);
}

// Cyclic reduction keeps about 5 b^2 words per layer of width b and applies them in
// 2 log2(layers) + 1 launches; block LU keeps 3 b^2 and needs 2 layers - 1 launches.  With
// few thick layers (3D subdomains: 9 layers of 1,282 at 8^3, 17 of 4,866 at 16^3) each
// block-LU launch is large enough to stream at full rate and block LU reads fewer bytes for
// the same K^{-1}; with many thin layers (2D meshes) the launches are latency-bound and the
// long chain of pivots is the less accurate one in FP32, so cyclic reduction is the form that
// the layers of such a mesh are limited by (see setup_precond).
constexpr int LU_MIN_LAYER = 1024;
constexpr int LU_MAX_LAYERS = 64;
static bool lu_shape(const Layering &L) {
    int64_t wide = 0;
    for (int32_t b : L.bsize) wide = std::max<int64_t>(wide, b);
    return wide >= LU_MIN_LAYER && L.nlayers <= LU_MAX_LAYERS;
}

// Maps of the layered forms for one system (host lists and their device copies).
static void layer_maps(thm_system &S, hipStream_t st) {
    if (S.Lskel_dof.n) return;
    const Topo &t = S.topo;
    build_layer_maps(t, S.dir, S.L);
    S.Lskel_dof.upload(S.L.skel_dof, st);
    S.Lskel_pos.upload(S.L.skel_pos, st);
    // global DoF -> padded position in the skeleton work vectors (-1: interior)
    std::vector<int32_t> vpos(S.L.dof_pos.size(), -1);
    for (size_t g = 0; g < vpos.size(); ++g)
        if (S.L.dof_pos[g] >= 0) vpos[g] = S.L.skel_pos[S.L.dof_pos[g]];
    S.Ldof_pos.upload(vpos, st);
    // per cell: padded positions of its skeleton (non-interior) local DoFs
    const int ne = t.n_loc - t.n_int;
    std::vector<int32_t> cpos((size_t)t.n_cells * ne);
    for (int64_t c = 0; c < t.n_cells; ++c)
        for (int le = 0; le < ne; ++le) cpos[(size_t)c * ne + le] = vpos[t.cell_dofs[(size_t)c * t.n_loc + le]];
    S.Lcell_pos.upload(cpos, st);
    S.Lcond_ptr.upload(S.L.cond_ptr, st);
    S.Lcond_cell.upload(S.L.cond_cell, st);
    S.Lcond_loc.upload(S.L.cond_loc, st);
    THM_HIP(hipStreamSynchronize(st));
}

// Apply layout of a layered factor's matrices (see k_repack).
static void repack(Factor &f, hipStream_t st) {
    std::vector<RepackDesc> rd;
    auto add = [&](const Factor::Blk &b) {
        RepackDesc d{};
        d.src = f.mat.p + b.off;
        d.rows = b.rows;
        d.cols = b.cols;
        d.ld = b.ld;
        d.nseg = b.nseg;
        d.poff = b.poff;
        int c = 0;
        for (int q = 0; q < b.nseg; ++q) {
            d.seg_col[q] = c;
            d.seg_len[q] = f.bsize[b.seg_layer[q]];
            d.seg_pstart[q] = b.seg_pstart[q];
            c += d.seg_len[q];
        }
        rd.push_back(d);
    };
    for (auto &lev : f.fwd)
        for (auto &b : lev) add(b);
    for (auto &lev : f.bwd)
        for (auto &b : lev) add(b);
    for (auto &b : f.tops) add(b);
    f.matp.alloc(std::max<int64_t>(f.matp_elems, 1));
    f.matp32.alloc(std::max<int64_t>(f.matp_elems, 1));
    launch_repack(rd, f.matp.p, f.matp32.p, st);
    THM_HIP(hipStreamSynchronize(st));
    f.mat.release();
}

// Offsets of the apply matrices of a nested-dissection factor.
static void nd_offsets(NdForm &f) {
    f.elems = 0;
    f.fo.assign(f.plan->ph.size(), {});
    f.bo.assign(f.plan->ph.size(), {});
    for (size_t q = 0; q < f.plan->ph.size(); ++q)
        for (const NdNode &v : f.plan->ph[q].node) {
            f.fo[q].push_back(f.elems);
            f.elems += nd_fwd_elems(v);
            f.bo[q].push_back(f.elems);
            f.elems += nd_bwd_elems(v);
        }
}

// One factorisation to do: its form (offsets set), destination and inputs.
struct NdJob {
    NdForm *form;
    thm_system *rep;
    double *m64;  // null in every job of a batch that only probes the growth
    float *m32;
    const double *kcond;
};

// Numerical factorisation of a batch, one phase at a time over all of it: fronts, inverses of
// the own blocks, G and the Schur complements, apply matrices.  Bad pivots are reported in
// *status, those of probes in one word per job and phase.
static void factor_nd(const NdJob *jobs, size_t nj, int32_t *status, long long *growth, hipStream_t st) {
    size_t np = 0;
    for (size_t t = 0; t < nj; ++t) np = std::max(np, jobs[t].form->plan->ph.size());
    DBuf<GemmDesc> gscr;
    Sched gsched;
    DBuf<double> Fprev;                        // fronts of the phase below (their Schur complements)
    std::vector<int64_t> cprev(nj, 0);  // first child entry per factor
    DBuf<NdChild> child;
    for (size_t q = 0; q < np; ++q) {
        int64_t fe = 0, de = 0, ge = 0;
        for (size_t t = 0; t < nj; ++t) {
            const NdPlan &plan = *jobs[t].form->plan;
            if (q >= plan.ph.size()) continue;
            for (const NdNode &v : plan.ph[q].node) {
                fe += (int64_t)(v.b + v.c) * (v.b + v.c);
                de += (int64_t)v.b * v.b;
                ge += (int64_t)v.b * v.c;
            }
        }
        DBuf<double> F(std::max<int64_t>(fe, 1)), Di(std::max<int64_t>(de, 1)), G(std::max<int64_t>(ge, 1));
        std::vector<NdFront> h;
        std::vector<NdChild> hc;
        std::vector<int64_t> cnext(nj, 0);
        fe = de = ge = 0;
        for (size_t t = 0; t < nj; ++t) {
            const NdJob &job = jobs[t];
            const NdPlan &plan = *job.form->plan;
            const int ne = job.rep->topo.n_loc - job.rep->topo.n_int;
            cnext[t] = (int64_t)hc.size();
            if (q >= plan.ph.size()) continue;
            const NdPhase &ph = plan.ph[q];
            for (size_t v = 0; v < ph.node.size(); ++v) {
                const NdNode &x = ph.node[v];
                const int n = x.b + x.c;
                NdFront r{};
                r.F = F.p + fe;
                r.b = x.b;
                r.c = x.c;
                r.kc = ph.kc;
                if (q == 0) {
                    r.ncell = x.nch;
                    r.cell = plan.d_leaf_cell.p + x.ch0;
                    r.row = plan.d_leaf_row.p + (int64_t)x.ch0 * ne;
                    r.kcond = job.kcond;
                    r.ne = ne;
                } else {
                    r.cidx = plan.d_cidx.p + x.loff;
                    r.cnode = plan.d_cnode.p + x.loff;
                    r.child = child.p + cprev[t];
                }
                r.own = plan.d_skel_dof.p + x.pos0;
                r.dir = job.rep->dir_d.p;
                r.Dinv = Di.p + de;
                r.G = G.p + ge;
                r.m64 = job.m64;
                r.m32 = job.m32;
                r.growth = growth + ND_LEVELS * t + q;
                r.status = job.m64 ? status : status + ND_LEVELS * t + q;
                if (job.m64) {
                    r.fo = job.form->fo[q][v];
                    r.bo = job.form->bo[q][v];
                }
                h.push_back(r);
                hc.push_back({r.F + (int64_t)x.b * n + x.b, n, x.uoff});
                fe += (int64_t)n * n;
                de += (int64_t)x.b * x.b;
                ge += (int64_t)x.b * x.c;
            }
        }
        DBuf<NdFront> dh;
        dh.upload(h, st);
        if (q == 0) launch_nd_leaf(h, dh.p, st);
        else launch_nd_merge(h, dh.p, st);
        launch_nd_invert(h, dh.p, st);
        int64_t wide = 0, widep = 0;
        for (const NdFront &r : h)
            if (r.b > ND_INV_MAX) {
                wide += 2 * (int64_t)r.b * r.b;
                widep += 2 * (int64_t)r.b;
            }
        if (wide) {
            DBuf<double> work(wide);
            DBuf<int32_t> piv(widep);
            std::vector<InvDesc> jobs;
            int64_t o = 0, op = 0;
            for (const NdFront &r : h) {
                if (r.b <= ND_INV_MAX) continue;
                launch_nd_own(r.F, r.b + r.c, r.b, work.p + o, st);
                jobs.push_back({r.b, work.p + o, work.p + o + (int64_t)r.b * r.b, r.Dinv, piv.p + op, r.b, r.status});
                o += 2 * (int64_t)r.b * r.b;
                op += 2 * r.b;
            }
            launch_invert_blocked(jobs, st);
        }
        std::vector<GemmDesc> ga, gb;
        for (const NdFront &r : h) {
            if (!r.b || !r.c) continue;
            const int n = r.b + r.c;
            ga.push_back({r.c, r.b, r.b, 0, 0, r.F + (int64_t)r.b * n, r.Dinv, r.G, n, r.b, r.b, 1.0, 0.0});
            gb.push_back({r.c, r.c, r.b, 0, 0, r.G, r.F + r.b, r.F + (int64_t)r.b * n + r.b, r.b, n, n, -1.0, 1.0});
        }
        launch_gemm_batched(ga, st, gscr, gsched);
        THM_HIP(hipStreamSynchronize(st));
        launch_gemm_batched(gb, st, gscr, gsched);
        if (jobs[0].m64) launch_nd_pack(h, dh.p, st);
        else launch_nd_growth(h, dh.p, st);
        child.upload(hc, st);
        THM_HIP(hipStreamSynchronize(st));
        Fprev = std::move(F);
        cprev = cnext;
    }
}

// Factorise every job, in batches whose widest phase of fronts fits 8 GiB.  Returns the growth of
// probes (jobs without matrices), ND_LEVELS entries each: the largest |G| per phase where it is
// beyond ND_GROWTH[0], else 0; infinity where a pivot was zero or not finite.
static std::vector<double> factor_nd_all(std::vector<NdJob> &jobs, int32_t *status, hipStream_t st) {
    std::vector<double> h(ND_LEVELS * jobs.size(), 0.0);
    if (jobs.empty()) return h;
    const bool probe = !jobs[0].m64;
    DBuf<long long> growth(h.size());
    THM_HIP(hipMemsetAsync(growth.p, 0, sizeof(long long) * growth.n, st));
    DBuf<int32_t> bad(h.size());  // of probes
    THM_HIP(hipMemsetAsync(bad.p, 0, sizeof(int32_t) * bad.n, st));
    for (size_t t0 = 0; t0 < jobs.size();) {
        size_t t1 = t0;
        int64_t words = 0;
        while (t1 < jobs.size()) {
            int64_t most = 0;
            for (const NdPhase &ph : jobs[t1].form->plan->ph) {
                int64_t w = 0;
                for (const NdNode &v : ph.node) w += 2 * (int64_t)(v.b + v.c) * (v.b + v.c);
                most = std::max(most, w);
            }
            if (t1 > t0 && words + most > (int64_t(1) << 30)) break;
            words += most;
            ++t1;
        }
        factor_nd(jobs.data() + t0, t1 - t0, probe ? bad.p + ND_LEVELS * t0 : status, growth.p + ND_LEVELS * t0, st);
        t0 = t1;
    }
    std::vector<int32_t> hb(h.size());
    THM_HIP(hipMemcpyAsync(h.data(), growth.p, sizeof(double) * h.size(), hipMemcpyDeviceToHost, st));
    THM_HIP(hipMemcpyAsync(hb.data(), bad.p, sizeof(int32_t) * hb.size(), hipMemcpyDeviceToHost, st));
    THM_HIP(hipStreamSynchronize(st));
    for (size_t i = 0; i < h.size(); ++i)
        if (hb[i]) h[i] = HUGE_VAL;
    return h;
}

enum class Form { nd, bcr, lu };

// Nested dissection keeps O(N log N) words (2D) where the layered forms keep O(N^1.5), in about
// as few launches as cyclic reduction: 64^2 cells of degree 2, FP64, 7 M words in 5 launches
// against 49 M in 7; 8^3 of degree 1, 8 M in 5 against 38 M in 17.  Its fronts are also better
// conditioned (FP32 backward error on the 64^2 square 4e-7 against 1e-5).  The layered forms
// stay for THM_FACTOR_FORM=bcr|lu.
static Form factor_form() {
    if (const char *e = std::getenv("THM_FACTOR_FORM")) {
        const std::string v(e);
        if (v == "lu") return Form::lu;
        if (v == "bcr") return Form::bcr;
        fail(THM_EINVAL, "THM_FACTOR_FORM must be bcr or lu");
    }
    return Form::nd;
}

// The plan of a system's mesh that avoids the given levels (see NdPlan): one that the system keeps
// (plans depend on the mesh alone), one of another system of the batch on the same mesh, or a new one.
constexpr size_t ND_KEPT = 8;  // plans a system keeps; the first two, the default and the probe, stay
static std::shared_ptr<NdPlan> nd_plan(thm_system &S, const std::vector<thm_system *> &others, uint64_t avoid,
                                       uint32_t barred, hipStream_t st) {
    auto kept = [&](const thm_system &o) -> std::shared_ptr<NdPlan> {
        for (const auto &p : o.nd)
            if (p->avoid == avoid && p->barred == barred && p->matches(S.topo)) return p;
        return nullptr;
    };
    std::shared_ptr<NdPlan> p = kept(S);
    if (p) return p;
    for (size_t i = 0; i < others.size() && !p; ++i) p = kept(*others[i]);
    if (!p) {
        p = std::make_shared<NdPlan>();
        p->avoid = avoid;
        p->barred = barred;
        nd_build_plan(S.topo, *p, st);
    }
    if (S.nd.size() >= ND_KEPT) S.nd.erase(S.nd.begin() + 2);
    S.nd.push_back(p);
    return p;
}

// Nested-dissection factors of a set of systems.  Near a resonance of its boxes a factor is as
// inexact as its growth (32^2 cells of degree 1 with w L = 6.25, close to 2 pi: relative residual
// of K z = x in FP32 1.2e-3 with boxes of 8 x 8 cells, growth 15, and 4e-5 with boxes of 8 x 16;
// in FP64 1e-11 and 1e-12).  So the growth of every halving level is found first, by a
// factorisation with every level as a phase (narrow fronts: about a third of the time of the
// other), and the phases start where it is small.  A box can also be singular where larger and
// smaller ones are not.  What the probe finds above the deepest level with such a box is of no use,
// so that level is barred and the probe repeated without it, as long as some tree is left.  Its
// pivots are reported apart from status, which also holds what the condensation reported.
static void setup_nd(const std::vector<thm_system *> &reps, const std::vector<std::shared_ptr<Factor>> &facs,
                     const std::vector<DBuf<double>> &kcond, const std::vector<thm_system *> &all, int32_t *status,
                     hipStream_t st) {
    std::vector<uint64_t> avoid(facs.size(), 0);
    std::vector<uint32_t> barred(facs.size(), 0);
    std::vector<NdForm> probe(facs.size());
    std::vector<NdJob> jobs;
    std::vector<size_t> at;
    for (size_t g = 0; g < facs.size(); ++g) {
        facs[g]->nd.plan = nd_plan(*reps[g], all, 0, 0, st);
        if (facs[g]->nd.plan->ph.size() >= 2) at.push_back(g);  // a root alone has no G
    }
    while (!at.empty()) {
        jobs.clear();
        for (size_t g : at) {
            probe[g].plan = nd_plan(*reps[g], all, ND_PROBE, barred[g], st);
            jobs.push_back({&probe[g], reps[g], nullptr, nullptr, kcond[g].p});
        }
        const std::vector<double> growth = factor_nd_all(jobs, nullptr, st);
        std::vector<size_t> again;
        for (size_t t = 0; t < at.size(); ++t) {
            const size_t g = at[t];
            const NdPlan &p = *probe[g].plan;
            const double *v = growth.data() + ND_LEVELS * t;
            size_t deep = 0;  // phases run from the leaves up
            while (deep < p.ph.size() && std::isfinite(v[deep])) ++deep;
            if (deep < p.ph.size()) {
                const uint32_t without = barred[g] | uint32_t(1) << p.from[deep];
                if (std::getenv("THM_PROGRESS"))
                    std::fprintf(stderr, "[thm]   tree level %d: singular\n", p.from[deep]);
                if (nd_avoidable(without, p.levels)) {
                    barred[g] = without;
                    again.push_back(g);
                    continue;
                }
            }
            for (size_t q = 0; q < p.ph.size(); ++q) {
                uint64_t cls = 0;
                while (cls + 1 < ND_CLASSES && !(v[q] <= ND_GROWTH[cls])) ++cls;
                if (p.from[q] > 0 && p.from[q] < ND_LEVELS) avoid[g] |= cls << (2 * p.from[q]);
                if (std::getenv("THM_PROGRESS"))
                    std::fprintf(stderr, "[thm]   tree level %d: growth %.3g\n", p.from[q], v[q]);
            }
        }
        at = again;
    }
    jobs.clear();
    for (size_t g = 0; g < facs.size(); ++g) {
        Factor &f = *facs[g];
        if (avoid[g] || barred[g]) f.nd.plan = nd_plan(*reps[g], all, avoid[g], barred[g], st);
        nd_offsets(f.nd);
        f.matp_elems = f.nd.elems;
        f.matp.alloc(std::max<int64_t>(f.matp_elems, 1));
        f.matp32.alloc(std::max<int64_t>(f.matp_elems, 1));
        jobs.push_back({&f.nd, reps[g], f.matp.p, f.matp32.p, kcond[g].p});
    }
    factor_nd_all(jobs, status, st);
}

void setup_precond(const std::vector<thm_system *> &all, hipStream_t st, bool share) {
    std::vector<thm_system *> need;
    for (thm_system *s : all)
        if (!s->fac) need.push_back(s);
    if (need.empty()) return;
    const double t0 = now_ms();
    // a setup that fails half way leaves no factor behind
    struct Unfinished {
        std::vector<thm_system *> &sys;
        bool done = false;
        ~Unfinished() {
            if (!done)
                for (thm_system *s : sys) s->fac.reset();
        }
    } unfinished{need};
    // group identical systems
    std::vector<std::shared_ptr<Factor>> facs;
    std::vector<thm_system *> reps;
    for (thm_system *s : need) {
        bool found = false;
        if (share)
            for (size_t g = 0; g < reps.size() && !found; ++g)
                if (same_topology(*reps[g], *s) && same_values(*reps[g], *s, st)) {
                    s->fac = facs[g];
                    found = true;
                }
        if (found) continue;
        auto f = std::make_shared<Factor>();
        s->fac = f;
        facs.push_back(f);
        reps.push_back(s);
    }
    const Form form = factor_form();
    if (form != Form::nd)
        for (thm_system *s : need) layer_maps(*s, st);
    DBuf<int32_t> status(1);
    THM_HIP(hipMemsetAsync(status.p, 0, sizeof(int32_t), st));
    std::vector<Work> W(facs.size());
    std::vector<DBuf<double>> kconds(facs.size());
    int maxlev = 0, maxn_lu = 0;
    for (size_t g = 0; g < facs.size(); ++g) {
        thm_system &R = *reps[g];
        Factor &f = *facs[g];
        const Layering &L = R.L;
        const Topo &t = R.topo;
        f.nlayers = L.nlayers;
        f.bsize = L.bsize;
        f.boff = L.boff;
        f.pboff = L.pboff;
        f.sp = L.n_skel_pad;
        f.n_int = t.n_int;
        f.ne = t.n_loc - t.n_int;
        f.n_cells = t.n_cells;
        f.lu = form == Form::lu;
        if (form == Form::nd) {
            // meshes whose layers are too wide for the layered forms are refused as ever
            Factor lay;
            lay.nlayers = f.nlayers;
            lay.bsize = f.bsize;
            lay.pboff = f.pboff;
            if (lu_shape(L)) plan_lu(lay);
            else plan(lay);
        } else if (f.lu) {
            plan_lu(f);
            maxn_lu = std::max(maxn_lu, f.nlayers);
        } else {
            plan(f);
            maxlev = std::max(maxlev, (int)f.fwd.size());
        }
        W[g].rep = &R;
        W[g].f = &f;
        // condensation of cell interiors
        f.kiinv.alloc(std::max<int64_t>((int64_t)t.n_cells * t.n_int * t.n_int, 1));
        f.F.alloc(std::max<int64_t>((int64_t)t.n_cells * f.ne * t.n_int, 1));
        DBuf<double> &kcond = kconds[g];
        kcond.alloc((size_t)t.n_cells * f.ne * f.ne);
        launch_condense((int)t.n_cells, t.n_loc, t.n_int, R.kel.p, R.cell_dofs.p, R.dir_d.p, f.kiinv.p, f.F.p,
                        kcond.p, status.p, st);
        if (form == Form::nd) continue;
        // initial blocks D_k, Lo_k from the condensed element matrices
        W[g].D.alloc(L.sinv_total);
        W[g].Lo0.alloc(std::max<int64_t>(L.lf_total, 1));
        launch_fill(W[g].D.p, L.sinv_total, 0.0, st);
        launch_fill(W[g].Lo0.p, L.lf_total, 0.0, st);
        {
            DBuf<int64_t> ti;
            DBuf<int32_t> tk, tp, ts;
            ti.upload(L.tgt_index, st);
            tk.upload(L.tgt_kind, st);
            tp.upload(L.tgt_ptr, st);
            ts.upload(L.tgt_src, st);
            launch_tgt_gather((int64_t)L.tgt_index.size(), ti.p, tk.p, tp.p, ts.p, kcond.p, W[g].D.p, W[g].Lo0.p, st);
            DBuf<int32_t> skel, bs;
            DBuf<int64_t> bo, so;
            skel.upload(L.skel_dof, st);
            bs.upload(L.bsize, st);
            bo.upload(L.boff, st);
            so.upload(L.sinv_off, st);
            launch_dir_identity(L.n_skel, skel.p, R.dir_d.p, bo.p, so.p, bs.p, L.nlayers, W[g].D.p, st);
            THM_HIP(hipStreamSynchronize(st));
        }
        kcond.release();
        f.mat.alloc(std::max<int64_t>(f.mat_elems, 1));
        for (int k = 0; k < L.nlayers; ++k) W[g].pos.push_back(k);
    }
    if (form == Form::nd) setup_nd(reps, facs, kconds, all, status.p, st);
    kconds.clear();
    DBuf<GemmDesc> gscr;
    Sched gsched;
    auto run_gemms = [&](const std::vector<GemmDesc> &g) {
        if (g.empty()) return;
        launch_gemm_batched(g, st, gscr, gsched);
        THM_HIP(hipStreamSynchronize(st));
    };
    // inversion scratch
    auto invert = [&](std::vector<std::pair<const double *, std::pair<double *, int>>> jobs, const std::vector<int> &ns) {
        if (jobs.empty()) return;
        int64_t tot = 0, totp = 0;
        for (int n : ns) { tot += 2 * (int64_t)n * n; totp += 2 * n; }
        DBuf<double> work(std::max<int64_t>(tot, 1));
        DBuf<int32_t> piv(std::max<int64_t>(totp, 1));
        std::vector<InvDesc> d;
        int64_t o = 0, op = 0;
        for (size_t j = 0; j < jobs.size(); ++j) {
            const int n = ns[j];
            double *A = work.p + o, *Wb = work.p + o + (int64_t)n * n;
            THM_HIP(hipMemcpyAsync(A, jobs[j].first, sizeof(double) * n * n, hipMemcpyDeviceToDevice, st));
            d.push_back({n, A, Wb, jobs[j].second.first, piv.p + op, jobs[j].second.second, status.p});
            o += 2 * (int64_t)n * n;
            op += 2 * n;
        }
        launch_invert_blocked(d, st);
    };
    const bool progress = std::getenv("THM_PROGRESS") != nullptr;
    if (progress)
        std::fprintf(stderr, "[thm] preconditioner setup: %zu systems, %zu factors, %d levels, %.1f ms\n", need.size(),
                     facs.size(), maxlev, now_ms() - t0);
    for (int lev = 0; lev < maxlev; ++lev) {
        if (progress) std::fprintf(stderr, "[thm]   level %d at %.1f ms\n", lev, now_ms() - t0);
        std::vector<std::pair<const double *, std::pair<double *, int>>> jobs;
        std::vector<int> jn;
        std::vector<GemmDesc> gA, gB1, gB2;
        struct LoNew { Work *w; int layer; DBuf<double> buf; };
        std::vector<LoNew> lonew;
        // 1. inverses of the odd positions (into the first columns of their back-substitution blocks)
        for (Work &w : W) {
            Factor &f = *w.f;
            if (f.lu || lev >= (int)f.fwd.size()) continue;
            const auto &pos = f.level_pos[lev];
            for (int i = 1; i < (int)pos.size(); i += 2) {
                const Factor::Blk &b = f.bwd[lev][f.bk_at[lev].at(i)];
                jobs.push_back({w.d_ptr(pos[i]), {f.mat.p + b.off, b.cols}});
                jn.push_back(b.rows);
            }
        }
        invert(jobs, jn);
        // 2. Gm, Gp; 3. D updates and new couplings
        for (Work &w : W) {
            Factor &f = *w.f;
            if (f.lu || lev >= (int)f.fwd.size()) continue;
            const auto &pos = f.level_pos[lev];
            const int m = (int)pos.size();
            for (int i = 0; i < m; i += 2) {
                const Factor::Blk &fb = f.fwd[lev][f.fw_at[lev].at(i)];
                const int bq = f.bsize[pos[i]];
                double *Fw = f.mat.p + fb.off;
                int cofs = 0;
                if (i > 0) {
                    const int bl = f.bsize[pos[i - 1]];
                    const Factor::Blk &bkl = f.bwd[lev][f.bk_at[lev].at(i - 1)];
                    gA.push_back({bq, bl, bl, 0, 0, w.lo_ptr(pos[i]), f.mat.p + bkl.off, Fw, bl, bkl.cols, fb.cols,
                                  1.0, 0.0});
                    gB1.push_back({bq, bq, bl, 0, 1, Fw, w.lo_ptr(pos[i]), w.d_ptr(pos[i]), fb.cols, bl, bq, -1.0, 1.0});
                    if (i >= 2) {
                        const int bll = f.bsize[pos[i - 2]];
                        lonew.push_back({&w, pos[i], DBuf<double>((size_t)bq * bll)});
                        gB1.push_back({bq, bll, bl, 0, 0, Fw, w.lo_ptr(pos[i - 1]), lonew.back().buf.p, fb.cols, bll,
                                       bll, -1.0, 0.0});
                    }
                    cofs = bl;
                }
                if (i + 1 < m) {
                    const int br = f.bsize[pos[i + 1]];
                    const Factor::Blk &bkr = f.bwd[lev][f.bk_at[lev].at(i + 1)];
                    // Gp = Lo_{i+1}^T Dinv_{i+1}; Lo_{i+1} is br x bq
                    gA.push_back({bq, br, br, 1, 0, w.lo_ptr(pos[i + 1]), f.mat.p + bkr.off, Fw + cofs, bq, bkr.cols,
                                  fb.cols, 1.0, 0.0});
                    gB2.push_back({bq, bq, br, 0, 0, Fw + cofs, w.lo_ptr(pos[i + 1]), w.d_ptr(pos[i]), fb.cols, bq, bq,
                                   -1.0, 1.0});
                }
            }
        }
        run_gemms(gA);
        run_gemms(gB1);
        run_gemms(gB2);
        // 4. back-substitution couplings: -Gp_{p-1}^T and -Gm_{p+1}^T next to Dinv_p
        for (Work &w : W) {
            Factor &f = *w.f;
            if (f.lu || lev >= (int)f.fwd.size()) continue;
            const auto &pos = f.level_pos[lev];
            const int m = (int)pos.size();
            for (int i = 1; i < m; i += 2) {
                const Factor::Blk &b = f.bwd[lev][f.bk_at[lev].at(i)];
                const int bp = f.bsize[pos[i]], bl = f.bsize[pos[i - 1]];
                const Factor::Blk &fl = f.fwd[lev][f.fw_at[lev].at(i - 1)];
                const int lcofs = (i - 1 > 0) ? f.bsize[pos[i - 2]] : 0;  // Gp part of Fw_{i-1}
                launch_transpose(f.mat.p + fl.off + lcofs, bl, bp, fl.cols, f.mat.p + b.off + bp, b.cols, -1.0, st);
                if (i + 1 < m) {
                    const Factor::Blk &fr = f.fwd[lev][f.fw_at[lev].at(i + 1)];
                    const int br = f.bsize[pos[i + 1]];
                    launch_transpose(f.mat.p + fr.off, br, bp, fr.cols, f.mat.p + b.off + bp + bl, b.cols, -1.0, st);
                }
            }
        }
        THM_HIP(hipStreamSynchronize(st));
        for (LoNew &ln : lonew) ln.w->lo[ln.layer] = std::move(ln.buf);
    }
    // block LU, one layer at a time over every block-LU factor
    for (int i = 0; i < maxn_lu; ++i) {
        if (progress) std::fprintf(stderr, "[thm]   block-LU layer %d at %.1f ms\n", i, now_ms() - t0);
        std::vector<GemmDesc> ga, gb, gd;
        std::vector<std::pair<const double *, std::pair<double *, int>>> jobs;
        std::vector<int> jn;
        for (Work &w : W) {
            Factor &f = *w.f;
            if (!f.lu || i >= f.nlayers || i == 0) continue;
            const int b = f.bsize[i], bl = f.bsize[i - 1];
            const Factor::Blk &fl = f.fwd[i - 1][0], &bk = f.bwd[i - 1][0];
            // backward matrix of layer i-1: S_{i-1}^{-1} Lo_i^T (Lo_i is b x bl)
            ga.push_back({bl, b, bl, 0, 1, f.mat.p + fl.off, w.lo_ptr(i), f.mat.p + bk.off, fl.cols, bl, b, 1.0, 0.0});
            // pivot S_i = D_i - Lo_i (S_{i-1}^{-1} Lo_i^T)
            gb.push_back({b, b, bl, 0, 0, w.lo_ptr(i), f.mat.p + bk.off, w.d_ptr(i), bl, b, b, -1.0, 1.0});
        }
        run_gemms(ga);
        run_gemms(gb);
        for (Work &w : W) {
            Factor &f = *w.f;
            if (!f.lu || i >= f.nlayers) continue;
            const Factor::Blk &fb = f.fwd[i][0];
            jobs.push_back({w.d_ptr(i), {f.mat.p + fb.off, fb.cols}});
            jn.push_back(fb.rows);
        }
        invert(jobs, jn);
        THM_HIP(hipStreamSynchronize(st));
        for (Work &w : W) {
            Factor &f = *w.f;
            if (!f.lu || i >= f.nlayers || i == 0) continue;
            const int b = f.bsize[i], bl = f.bsize[i - 1];
            const Factor::Blk &fb = f.fwd[i][0];
            // second block of the forward matrix: -S_i^{-1} Lo_i
            gd.push_back({b, bl, b, 0, 0, f.mat.p + fb.off, w.lo_ptr(i), f.mat.p + fb.off + b, fb.cols, bl, fb.cols,
                          -1.0, 0.0});
        }
        run_gemms(gd);
    }
    // last blocks: assemble the remaining block-tridiagonal system densely and invert it
    {
        std::vector<std::pair<const double *, std::pair<double *, int>>> jobs;
        std::vector<int> jn;
        std::vector<DBuf<double>> dense(W.size());
        for (size_t g = 0; g < W.size(); ++g) {
            Work &w = W[g];
            Factor &f = *w.f;
            if (f.lu || f.nd.plan) continue;
            const int N = f.top_n;
            dense[g].alloc((size_t)N * N);
            launch_fill(dense[g].p, (int64_t)N * N, 0.0, st);
            int64_t ro = 0;
            std::vector<int64_t> offs;
            for (int k : f.top_pos) {
                offs.push_back(ro);
                ro += f.bsize[k];
            }
            for (size_t i = 0; i < f.top_pos.size(); ++i) {
                const int k = f.top_pos[i], b = f.bsize[k];
                double *blk = dense[g].p + offs[i] * N + offs[i];
                THM_HIP(hipMemcpy2DAsync(blk, sizeof(double) * N, w.d_ptr(k), sizeof(double) * b, sizeof(double) * b,
                                         b, hipMemcpyDeviceToDevice, st));
                if (i > 0) {
                    const int kl = f.top_pos[i - 1], bl = f.bsize[kl];
                    // T[i][i-1] = Lo (b x bl), T[i-1][i] = Lo^T
                    THM_HIP(hipMemcpy2DAsync(dense[g].p + offs[i] * N + offs[i - 1], sizeof(double) * N,
                                             w.lo_ptr(k), sizeof(double) * bl, sizeof(double) * bl, b,
                                             hipMemcpyDeviceToDevice, st));
                    launch_transpose(w.lo_ptr(k), b, bl, bl, dense[g].p + offs[i - 1] * N + offs[i], N, 1.0, st);
                }
            }
            jobs.push_back({dense[g].p, {f.mat.p + f.top_off, N}});
            jn.push_back(N);
        }
        THM_HIP(hipStreamSynchronize(st));
        invert(jobs, jn);
    }
    for (Work &w : W) {
        Factor &f = *w.f;
        if (!f.nd.plan) repack(f, st);
        // apply layouts: K_ii^{-1} transposed per cell, F and F^T
        if (f.n_int > 0) {
            DBuf<double> kt(f.kiinv.n);
            launch_batch_transpose(f.n_cells, f.n_int, f.n_int, f.kiinv.p, kt.p, st);
            THM_HIP(hipMemcpyAsync(f.kiinv.p, kt.p, sizeof(double) * kt.n, hipMemcpyDeviceToDevice, st));
            THM_HIP(hipStreamSynchronize(st));
        }
        f.FT.alloc(f.F.n);
        launch_batch_transpose(f.n_int > 0 ? f.n_cells : 0, f.ne, f.n_int, f.F.p, f.FT.p, st);
        f.kiinv32.alloc(f.kiinv.n);
        f.F32.alloc(f.F.n);
        f.FT32.alloc(f.F.n);
        launch_convert(f.kiinv.p, f.kiinv32.p, f.kiinv.n, st);
        launch_convert(f.F.p, f.F32.p, f.F.n, st);
        launch_convert(f.FT.p, f.FT32.p, f.FT.n, st);
        w.D.release();
        w.Lo0.release();
        w.lo.clear();
    }
    int32_t hs = 0;
    THM_HIP(hipMemcpyAsync(&hs, status.p, sizeof(int32_t), hipMemcpyDeviceToHost, st));
    THM_HIP(hipStreamSynchronize(st));
    if (hs) fail(THM_ESINGULAR, "zero or non-finite pivot while factorising the block preconditioner");
    const double dt = now_ms() - t0;
    for (auto &f : facs) {
        f->setup_ms = dt;
        f->bytes = 12 * (f->matp_elems + (int64_t)f->kiinv.n + 2 * (int64_t)f->F.n);
    }
    unfinished.done = true;
}

}  // namespace thm
