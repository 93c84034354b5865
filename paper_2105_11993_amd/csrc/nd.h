// Nested-dissection form of the exact K^{-1}: the plan (host, integer bookkeeping), and the
// launchers of its factorisation and application (kernels_nd.hip).
//
// The box of cells is halved along its longest axis until at most ND_LEAF cells remain.  A
// skeleton DoF belongs to the deepest box that contains every cell it touches.  Consecutive
// halving levels are merged into a few phases; a node of a phase is one box at the phase's
// first level, its own DoFs are those of the levels the phase covers, and its boundary are the
// DoFs of the box that belong to higher phases.  Phases run from the leaves (phase 0) to the
// root (one node without boundary).  With F the node's dense front on [own; boundary],
//   Dinv = F_oo^{-1},  G = F_bo Dinv,  U = F_bb - G F_ob  (added into the parent's front),
// and one application is, up the tree, u = (children's u on the boundary) + G r with
// r = rhs - (children's u on the own DoFs), and down the tree x = Dinv r - G^T x_boundary.
#pragma once
#include "thm_internal.h"
#include "kernels.h"

namespace thm {

constexpr int ND_LEAF = 4;      // cells of a box that is not halved any further
constexpr int ND_MERGE = 6;     // halving levels one phase may cover
constexpr int ND_RT = 16;       // rows of a matrix tile
constexpr int ND_KS = 16;       // columns are padded to this
// A node whose box is close to a resonance of its own (its F_oo nearly singular) has a large G,
// and its rounding errors grow with it; entries of G stay near 1 to 2 otherwise.  Levels are
// classed by their largest entry: 0 up to ND_GROWTH[0], 1 up to ND_GROWTH[1] and so on.
constexpr int ND_CLASSES = 4;
constexpr double ND_GROWTH[ND_CLASSES - 1] = {3.0, 12.0, 100.0};
constexpr int ND_LEVELS = 32;

struct NdNode {
    int32_t b, c;       // own DoFs, boundary DoFs
    int32_t pos0;       // first own position
    int32_t uoff;       // first boundary entry (in bpos and in the update vector)
    int32_t ch0, nch;   // children: nodes [ch0, ch0 + nch) of the phase below (phase 0: cells, in leaf_cell)
    int64_t loff;       // first entry of the front's child lists ((b + c) x kc, phases above 0)
};

struct NdPhase {
    int kc = 0;                 // update rows gathered per front row at most
    std::vector<NdNode> node;
};

struct NdPlan {
    int dim = 0, p = 0, n[3] = {0, 0, 0};
    int64_t n_skel = 0, n_upd = 0;
    // class of every halving level as the start of a phase (two bits each); ND_PROBE: every
    // level is a phase, but for those in barred
    uint64_t avoid = 0;
    uint32_t barred = 0;        // levels (bit each) where some box is singular
    int levels = 0;             // halving levels
    std::vector<int> from;      // first level of each phase
    std::vector<NdPhase> ph;    // leaves first
    std::vector<int32_t> skel_dof;   // position -> DoF
    std::vector<int32_t> bpos;       // boundary entry -> position
    std::vector<int32_t> cidx;       // child lists: update entry, -1 none
    std::vector<int32_t> cnode;      // child lists: node of the phase below
    std::vector<int32_t> leaf_cell;  // cells of the leaves, by NdNode::ch0
    std::vector<int32_t> leaf_row;   // per leaf_cell entry: front row of each skeleton local DoF
    // device copies
    DBuf<int32_t> d_skel_dof, d_bpos, d_cidx, d_cnode, d_leaf_cell, d_leaf_row;
    DBuf<int32_t> d_dof_pos, d_cell_pos, d_cond_ptr, d_cond_cell, d_cond_loc;
    bool matches(const Topo &t) const {
        return dim == t.dim && p == t.p && n[0] == t.n[0] && n[1] == t.n[1] && n[2] == t.n[2];
    }
};

// A factorisation on a plan: per phase and node the offsets of its two apply matrices.
struct NdForm {
    std::shared_ptr<NdPlan> plan;
    std::vector<std::vector<int64_t>> fo, bo;
    int64_t elems = 0;
};

constexpr uint64_t ND_PROBE = ~uint64_t(0);
// Some tree starts no phase at the levels in barred: they are no run of ND_MERGE or more.
bool nd_avoidable(uint32_t barred, int levels);
void nd_plan_mesh(const Topo &t, NdPlan &P);                     // host part
void nd_build_plan(const Topo &t, NdPlan &P, hipStream_t st);    // with the device copies

// Padded element counts of a node's apply matrices: G (c x b), then [Dinv | -G^T] (b x (b + c)).
__host__ __device__ inline int64_t nd_pad(int64_t v, int64_t a) { return (v + a - 1) / a * a; }
inline int64_t nd_fwd_elems(const NdNode &v) { return nd_pad(v.c, ND_RT) * nd_pad(v.b, ND_KS); }
inline int64_t nd_bwd_elems(const NdNode &v) { return nd_pad(v.b, ND_RT) * nd_pad(v.b + v.c, ND_KS); }

// ---- factorisation
struct NdChild {        // a node of the phase below as seen by the front assembly
    const double *U;    // its Schur complement, leading dimension ld
    int32_t ld, uoff;
};
struct NdFront {
    double *F;                  // n x n front, n = b + c
    int32_t b, c, kc, ncell, ne;    // ne: skeleton DoFs of a cell
    const int32_t *cidx, *cnode;    // child lists of the node (phases above 0)
    const NdChild *child;           // the phase below, all nodes of this factor
    const int32_t *cell, *row;      // phase 0: cells and their front rows
    const double *kcond;            // phase 0: condensed element matrices
    const int32_t *own;             // own DoFs
    const uint8_t *dir;             // Dirichlet flags (their rows become the identity)
    double *Dinv, *G;               // results: b x b, c x b
    long long *growth;              // largest |G| of the phase beyond ND_GROWTH[0], as bits (NaN as infinity)
    int32_t *status;                // |= 1 for a zero or non-finite pivot
    double *m64;                    // apply matrices, FP64 and FP32
    float *m32;
    int64_t fo, bo;                 // element offsets of the two apply matrices
};
void launch_nd_leaf(const std::vector<NdFront> &h, const NdFront *d, hipStream_t st);
void launch_nd_merge(const std::vector<NdFront> &h, const NdFront *d, hipStream_t st);
// Dinv = F_oo^{-1} for the fronts with 0 < b <= ND_INV_MAX (one workgroup each, partial pivoting)
constexpr int ND_INV_MAX = 128;
void launch_nd_invert(const std::vector<NdFront> &h, const NdFront *d, hipStream_t st);
// A = F_oo as a contiguous matrix
void launch_nd_own(const double *F, int n, int b, double *A, hipStream_t st);
void launch_nd_growth(const std::vector<NdFront> &h, const NdFront *d, hipStream_t st);
void launch_nd_pack(const std::vector<NdFront> &h, const NdFront *d, hipStream_t st);

// ---- application
// Blocks of one launch: some row tiles of one node for some members of its factor group.
struct NdTask {
    const void *M;              // tile-ordered matrix
    const int32_t *bpos, *cidx; // boundary positions of the node; its child lists
    int64_t gbase, ubase;       // the group's start in ws / ys and in the update vector
    int32_t b, c, pos0, uoff;
    int32_t cs;                 // scalars per position: 2 x members of the group
    int32_t mbeg, m0, nm;       // members [m0, m0 + nm) of the group, whose list starts at mbeg
    int32_t rt0, tiles;         // row tiles of the block
    int16_t kc, ks;             // child lists per row; waves sharing a row tile
};
constexpr int ND_KC_VEC = 2048;  // columns staged at a time, one member
struct NdLaunch {
    bool fwd = true, vec = true;    // vec: groups of one member
    int nblocks = 0, waves = 4;     // waves of a block: 4 or 8
    size_t lds = 0;
    DBuf<NdTask> tasks;
};
template <class T>
void launch_nd_phases(const std::vector<NdLaunch> &L, const int32_t *memb, const int32_t *mask, const T *ws, T *ys,
                      T *ub, hipStream_t st);

}  // namespace thm
