// Plan of the nested-dissection form of K^{-1} (see nd.h): integer bookkeeping on the mesh
// entities (edges and faces), expanded to DoFs.
#include <algorithm>

#include "nd.h"

namespace thm {

namespace {

struct Box {
    int lo[3], hi[3];
    int64_t cells() const { return (int64_t)(hi[0] - lo[0]) * (hi[1] - lo[1]) * (hi[2] - lo[2]); }
};

// Mesh entities carrying skeleton DoFs: first DoF, DoF count, touching cells (-1: none).
struct Entity {
    int32_t dof, w;
    int32_t cell[4];
};

std::vector<Entity> entities(const Topo &t) {
    std::vector<Entity> out;
    auto cell = [&](int i, int j, int k) -> int32_t {
        if (i < 0 || j < 0 || k < 0 || i >= t.n[0] || j >= t.n[1] || k >= t.n[2]) return -1;
        return (int32_t)(((int64_t)k * t.n[1] + j) * t.n[0] + i);
    };
    auto family = [&](const int *odd, int64_t off, int w) {  // odd[a]: the entity spans a cell along axis a
        int size[3];
        for (int a = 0; a < 3; ++a) size[a] = a < t.dim ? t.n[a] + (odd[a] ? 0 : 1) : 1;
        int32_t id = 0;
        for (int k = 0; k < size[2]; ++k)
            for (int j = 0; j < size[1]; ++j)
                for (int i = 0; i < size[0]; ++i, ++id) {
                    Entity e;
                    e.dof = (int32_t)(off + (int64_t)id * w);
                    e.w = w;
                    int m = 0;
                    for (int dk = (odd[2] || t.dim < 3) ? 0 : -1; dk <= 0; ++dk)
                        for (int dj = odd[1] ? 0 : -1; dj <= 0; ++dj)
                            for (int di = odd[0] ? 0 : -1; di <= 0; ++di) {
                                const int32_t c = cell(i + di, j + dj, k + dk);
                                if (c >= 0) e.cell[m++] = c;
                            }
                    for (; m < 4; ++m) e.cell[m] = -1;
                    out.push_back(e);
                }
    };
    for (int a = 0; a < t.dim; ++a) {
        const int odd[3] = {a == 0, a == 1, a == 2};
        family(odd, t.edge_off[a], t.pe);
    }
    if (t.dim == 3 && t.pf > 0)
        for (int a = 0; a < 3; ++a) {
            const int odd[3] = {a != 0, a != 1, a != 2};
            family(odd, t.face_off[a], t.pf);
        }
    return out;
}

// Estimated seconds of one application and of the factorisation, for the choice of phases: a
// launch takes about 6 us in a replayed graph where its matrices are small (64^2 cells of degree
// 2: 4.8 to 7 us for phases of 2 to 10 MB), the matrices stream at about 5 TB/s (62 MB in 14 us, 479
// in 88), and the factorisation (2 us per column of the widest front, FP64 products at 10
// TFLOP/s) is shared by about 200 applications, one or two solves.
constexpr double ND_LAUNCH_S = 6e-6, ND_BYTES_S = 5e12, ND_COL_S = 2e-6, ND_FLOP_S = 1e13, ND_REUSE = 200;
// What a level that a phase starts at adds to the cost, by its class, as a part of the cheapest
// plan's seconds: the errors of such levels multiply, and an FP32 solve takes more refinement steps
// or has to be finished in FP64.  (16^3 cells of degree 1 at w = 15, growth 20 to 190 on every
// level: 8 levels started at 364 us an application, 5 in 486 us; a mixed solve 220 and 175 ms.)
constexpr double ND_CLASS_COST[ND_CLASSES] = {0.0, 0.33, 0.6, 3.0};
// The same for a level with a singular box: any tree without it is cheaper.
constexpr double ND_BARRED_COST = 1e6;

}  // namespace

bool nd_avoidable(uint32_t barred, int levels) {
    if (barred & 1u) return false;  // the root
    for (int l = 0, run = 0; l < levels; ++l) {
        run = (barred >> l) & 1u ? run + 1 : 0;
        if (run >= ND_MERGE) return false;
    }
    return true;
}

void nd_plan_mesh(const Topo &t, NdPlan &P) {
    P.dim = t.dim;
    P.p = t.p;
    std::copy(t.n, t.n + 3, P.n);
    P.n_skel = t.cell_off;
    // halving levels: the box of every cell, boxes of a level in order so that the parts of a
    // box stay consecutive
    std::vector<std::vector<int32_t>> id;      // [level][cell]
    std::vector<std::vector<int32_t>> first;   // [level][box]: first box of the next level inside it
    std::vector<int> nbox;
    std::vector<Box> boxes(1);
    for (int a = 0; a < 3; ++a) {
        boxes[0].lo[a] = 0;
        boxes[0].hi[a] = t.n[a];
    }
    for (;;) {
        std::vector<int32_t> g(t.n_cells);
        for (size_t q = 0; q < boxes.size(); ++q)
            for (int k = boxes[q].lo[2]; k < boxes[q].hi[2]; ++k)
                for (int j = boxes[q].lo[1]; j < boxes[q].hi[1]; ++j)
                    for (int i = boxes[q].lo[0]; i < boxes[q].hi[0]; ++i)
                        g[((int64_t)k * t.n[1] + j) * t.n[0] + i] = (int32_t)q;
        id.push_back(std::move(g));
        nbox.push_back((int)boxes.size());
        std::vector<Box> next;
        std::vector<int32_t> f;
        for (const Box &x : boxes) {
            f.push_back((int32_t)next.size());
            if (x.cells() <= ND_LEAF) {
                next.push_back(x);
                continue;
            }
            int a = 0;
            for (int q = 1; q < 3; ++q)
                if (x.hi[q] - x.lo[q] > x.hi[a] - x.lo[a]) a = q;
            const int m = (x.lo[a] + x.hi[a]) / 2;
            Box l = x, r = x;
            l.hi[a] = m;
            r.lo[a] = m;
            next.push_back(l);
            next.push_back(r);
        }
        f.push_back((int32_t)next.size());
        if (next.size() == boxes.size()) break;
        first.push_back(std::move(f));
        boxes = std::move(next);
    }
    const int D = (int)id.size();
    // level of every entity (deepest level at which one box holds all its cells), and per
    // level and box the DoFs by entity level
    const std::vector<Entity> ents = entities(t);
    const size_t ne = ents.size();
    std::vector<int> lev(ne, 0);
    std::vector<std::vector<int32_t>> hist(D);  // [level][box * D + entity level]
    for (int l = 0; l < D; ++l) hist[l].assign((size_t)nbox[l] * D, 0);
    auto boxes_of = [&](const Entity &e, int l, int32_t *out) {  // distinct boxes touched at level l
        int m = 0;
        for (int q = 0; q < 4 && e.cell[q] >= 0; ++q) {
            const int32_t b = id[l][e.cell[q]];
            bool seen = false;
            for (int r = 0; r < m; ++r) seen = seen || out[r] == b;
            if (!seen) out[m++] = b;
        }
        return m;
    };
    for (size_t e = 0; e < ne; ++e) {
        int32_t bx[4];
        int l = 0;
        while (l + 1 < D && boxes_of(ents[e], l + 1, bx) == 1) ++l;
        lev[e] = l;
        for (int q = 0; q < D; ++q) {
            const int m = boxes_of(ents[e], q, bx);
            for (int r = 0; r < m; ++r) hist[q][(size_t)bx[r] * D + l] += ents[e].w;
        }
    }
    // phases: cheapest split of the levels, from the root down
    std::vector<std::vector<double>> seconds(D, std::vector<double>(D + 1, 0.0));  // of a phase [a, z)
    for (int a = 0; a < D; ++a) {
        std::vector<int64_t> own(nbox[a], 0), bnd(nbox[a], 0);
        for (int q = 0; q < nbox[a]; ++q)
            for (int l = 0; l < a; ++l) bnd[q] += hist[a][(size_t)q * D + l];
        for (int z = a + 1; z <= std::min(D, a + ND_MERGE); ++z) {
            double words = 0.0, flops = 0.0, wide = 0.0;
            for (int q = 0; q < nbox[a]; ++q) {
                own[q] += hist[a][(size_t)q * D + z - 1];
                const double b = (double)own[q], c = (double)bnd[q];
                words += b * b + 2.0 * b * c;
                flops += 2.0 * b * b * b + 2.0 * b * b * c + 2.0 * b * c * c;
                wide = std::max(wide, b);
            }
            seconds[a][z] = (a > 0 ? 2.0 : 1.0) * ND_LAUNCH_S + 8.0 * words / ND_BYTES_S +
                            (wide * ND_COL_S + flops / ND_FLOP_S) / ND_REUSE;
        }
    }
    auto is_barred = [&](int a) { return a > 0 && a < ND_LEVELS && ((P.barred >> a) & 1u); };
    auto level_cost = [&](int a) {
        if (is_barred(a)) return ND_BARRED_COST;
        return ND_CLASS_COST[a > 0 && a < ND_LEVELS ? (P.avoid >> (2 * a)) & 3u : 0];
    };
    std::vector<int> cut(D + 1, D);
    double least = 0.0;  // seconds of the cheapest plan, whatever its levels
    for (bool weigh : {false, true}) {
        std::vector<double> best(D + 1, -1.0);
        best[D] = 0.0;
        for (int a = D - 1; a >= 0; --a)
            for (int z = a + 1; z <= std::min(D, a + ND_MERGE); ++z) {
                const double s = seconds[a][z] + best[z] + (weigh ? level_cost(a) * least : 0.0);
                if (best[a] < 0.0 || s < best[a]) {
                    best[a] = s;
                    cut[a] = z;
                }
            }
        least = best[0];
        if ((!P.avoid && !P.barred) || P.avoid == ND_PROBE) break;
    }
    std::vector<int> from;  // first level of each phase, root first
    if (P.avoid == ND_PROBE) {
        for (int a = 0; a < D; ++a)
            if (!is_barred(a)) from.push_back(a);
    } else {
        for (int a = 0; a < D; a = cut[a]) from.push_back(a);
    }
    const int np = (int)from.size();
    std::reverse(from.begin(), from.end());  // leaves first
    std::vector<int> phase_of(D);
    for (int l = 0; l < D; ++l) {
        int f = 0;
        while (f + 1 < np && from[f] > l) ++f;
        phase_of[l] = f;
    }
    P.from = from;
    P.levels = D;
    // own entities per node, deeper levels first; positions in elimination order
    P.ph.assign(np, NdPhase());
    std::vector<std::vector<std::vector<int32_t>>> own(np), bnd(np);
    for (int f = 0; f < np; ++f) {
        own[f].resize(nbox[from[f]]);
        bnd[f].resize(nbox[from[f]]);
        P.ph[f].node.assign(nbox[from[f]], NdNode{});
    }
    {
        std::vector<std::vector<int32_t>> by(D);
        for (size_t e = 0; e < ne; ++e) by[lev[e]].push_back((int32_t)e);
        for (int l = D - 1; l >= 0; --l)
            for (int32_t e : by[l]) own[phase_of[l]][id[from[phase_of[l]]][ents[e].cell[0]]].push_back(e);
    }
    std::vector<int32_t> epos(ne, 0);
    P.skel_dof.assign(P.n_skel, 0);
    std::vector<int32_t> order;  // entities by position
    order.reserve(ne);
    int32_t pos = 0;
    for (int f = 0; f < np; ++f)
        for (size_t q = 0; q < own[f].size(); ++q) {
            NdNode &v = P.ph[f].node[q];
            v.pos0 = pos;
            for (int32_t e : own[f][q]) {
                epos[e] = pos;
                order.push_back(e);
                for (int32_t i = 0; i < ents[e].w; ++i) P.skel_dof[pos++] = ents[e].dof + i;
            }
            v.b = pos - v.pos0;
        }
    for (int32_t e : order) {  // ascending positions
        const int pe = phase_of[lev[e]];
        int32_t bx[4];
        for (int f = 0; f < pe; ++f) {
            const int m = boxes_of(ents[e], from[f], bx);
            for (int r = 0; r < m; ++r) bnd[f][bx[r]].push_back(e);
        }
    }
    int64_t uo = 0;
    P.bpos.clear();
    for (int f = 0; f < np; ++f)
        for (size_t q = 0; q < bnd[f].size(); ++q) {
            NdNode &v = P.ph[f].node[q];
            v.uoff = (int32_t)uo;
            for (int32_t e : bnd[f][q])
                for (int32_t i = 0; i < ents[e].w; ++i) P.bpos.push_back(epos[e] + i);
            uo = (int64_t)P.bpos.size();
            if (uo > INT32_MAX) fail(THM_EUNSUPPORTED, "mesh too large for 32-bit update indices");
            v.c = (int32_t)(uo - v.uoff);
        }
    P.n_upd = uo;
    // children: leaves hold cells, other nodes the boxes of the phase below
    const int nl = t.n_loc, nsk = t.n_loc - t.n_int;
    std::vector<int32_t> row(ne, -1);  // front row of an entity in the node at hand
    auto set_rows = [&](int f, size_t q) {
        int32_t r = 0;
        for (int32_t e : own[f][q]) {
            row[e] = r;
            r += ents[e].w;
        }
        for (int32_t e : bnd[f][q]) {
            row[e] = r;
            r += ents[e].w;
        }
    };
    {
        std::vector<std::vector<int32_t>> cells(nbox[from[0]]);
        for (int64_t c = 0; c < t.n_cells; ++c) cells[id[from[0]][c]].push_back((int32_t)c);
        std::vector<int32_t> ent_of(P.n_skel);  // DoF -> entity
        for (size_t e = 0; e < ne; ++e)
            for (int32_t i = 0; i < ents[e].w; ++i) ent_of[ents[e].dof + i] = (int32_t)e;
        P.leaf_cell.clear();
        P.leaf_row.clear();
        for (size_t q = 0; q < cells.size(); ++q) {
            NdNode &v = P.ph[0].node[q];
            v.ch0 = (int32_t)P.leaf_cell.size();
            v.nch = (int32_t)cells[q].size();
            set_rows(0, q);
            for (int32_t c : cells[q]) {
                P.leaf_cell.push_back(c);
                for (int u = 0; u < nsk; ++u) {
                    const int32_t g = t.cell_dofs[(size_t)c * nl + u], e = ent_of[g];
                    P.leaf_row.push_back(row[e] + (g - ents[e].dof));
                }
            }
        }
    }
    P.cidx.clear();
    P.cnode.clear();
    for (int f = 1; f < np; ++f) {
        NdPhase &ph = P.ph[f];
        std::vector<int32_t> cnt;
        // children of box q: the boxes of the phase below inside it
        for (size_t q = 0; q < ph.node.size(); ++q) {
            int32_t c0 = (int32_t)q, c1 = (int32_t)q + 1;
            for (int l = from[f]; l < from[f - 1]; ++l) {
                c0 = first[l][c0];
                c1 = first[l][c1];
            }
            ph.node[q].ch0 = c0;
            ph.node[q].nch = c1 - c0;
        }
        auto each = [&](auto put) {  // every (node, front row, child, child's update entry)
            for (size_t q = 0; q < ph.node.size(); ++q) {
                const NdNode &v = ph.node[q];
                set_rows(f, q);
                for (int32_t ch = v.ch0; ch < v.ch0 + v.nch; ++ch) {
                    int32_t u = P.ph[f - 1].node[ch].uoff;
                    for (int32_t e : bnd[f - 1][ch])
                        for (int32_t i = 0; i < ents[e].w; ++i) put(q, row[e] + i, ch, u++);
                }
            }
        };
        std::vector<int64_t> fo(ph.node.size() + 1, 0);
        for (size_t q = 0; q < ph.node.size(); ++q) fo[q + 1] = fo[q] + ph.node[q].b + ph.node[q].c;
        cnt.assign(fo.back(), 0);
        each([&](size_t q, int32_t r, int32_t, int32_t) { ++cnt[fo[q] + r]; });
        ph.kc = 1;
        for (int32_t v : cnt) ph.kc = std::max(ph.kc, (int)v);
        if (ph.kc == 3) ph.kc = 4;
        if (ph.kc > 4) fail(THM_EINVAL, "internal: a skeleton DoF touches more than four boxes");
        const int64_t base = (int64_t)P.cidx.size();
        P.cidx.resize(base + fo.back() * ph.kc, -1);
        P.cnode.resize(base + fo.back() * ph.kc, -1);
        for (size_t q = 0; q < ph.node.size(); ++q) ph.node[q].loff = base + fo[q] * ph.kc;
        std::fill(cnt.begin(), cnt.end(), 0);
        each([&](size_t q, int32_t r, int32_t ch, int32_t u) {
            const int64_t s = base + (fo[q] + r) * ph.kc + cnt[fo[q] + r]++;
            P.cidx[s] = u;
            P.cnode[s] = ch;
        });
    }
}

void nd_build_plan(const Topo &t, NdPlan &P, hipStream_t st) {
    nd_plan_mesh(t, P);
    const int nl = t.n_loc, nsk = t.n_loc - t.n_int;
    // device copies and the maps of the condensation kernels
    std::vector<int32_t> dof_pos(t.n_dofs, -1), cell_pos((size_t)t.n_cells * nsk);
    for (int64_t i = 0; i < P.n_skel; ++i) dof_pos[P.skel_dof[i]] = (int32_t)i;
    std::vector<int32_t> cptr(P.n_skel + 1, 0), ccell((size_t)t.n_cells * nsk), cloc(ccell.size());
    for (int64_t c = 0; c < t.n_cells; ++c)
        for (int u = 0; u < nsk; ++u) {
            const int32_t q = dof_pos[t.cell_dofs[(size_t)c * nl + u]];
            cell_pos[(size_t)c * nsk + u] = q;
            cptr[q + 1]++;
        }
    for (int64_t i = 0; i < P.n_skel; ++i) cptr[i + 1] += cptr[i];
    {
        std::vector<int32_t> fill(cptr.begin(), cptr.end() - 1);
        for (int64_t c = 0; c < t.n_cells; ++c)
            for (int u = 0; u < nsk; ++u) {
                const int32_t s = fill[cell_pos[(size_t)c * nsk + u]]++;
                ccell[s] = (int32_t)c;
                cloc[s] = u;
            }
    }
    P.d_skel_dof.upload(P.skel_dof, st);
    P.d_bpos.upload(P.bpos, st);
    P.d_cidx.upload(P.cidx, st);
    P.d_cnode.upload(P.cnode, st);
    P.d_leaf_cell.upload(P.leaf_cell, st);
    P.d_leaf_row.upload(P.leaf_row, st);
    P.d_dof_pos.upload(dof_pos, st);
    P.d_cell_pos.upload(cell_pos, st);
    P.d_cond_ptr.upload(cptr, st);
    P.d_cond_cell.upload(ccell, st);
    P.d_cond_loc.upload(cloc, st);
    THM_HIP(hipStreamSynchronize(st));  // the host copies of the last five end here
}

}  // namespace thm
