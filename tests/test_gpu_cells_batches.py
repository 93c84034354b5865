"""The product from the cells (SpMV code 30) where its launch takes other forms: groups of 1, 2, 9 and 16
members with partly filled last tiles and masked members, pinned through a tuning cache that a child
process reads; and a mesh of so many cells that a block takes several rounds of tiles.
"""
import os
import subprocess
import sys

import numpy as np
import pytest
import scipy.sparse as sp

from oracle import system
from tests._gpu_helpers import problem, rel, spec

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
# members and mesh: cells x members is no multiple of 8 but for 16; above the 3 million entries from which
# the cells are offered
GROUPS = {1: (77, 75), 2: (53, 53), 9: (25, 25), 16: (19, 20)}


def members(count):
    n = GROUPS[count]
    rng = np.random.default_rng(40 + count)
    mu, eps = rng.uniform(1.0, 2.0, n[0] * n[1]), rng.uniform(1.0, 1.5, n[0] * n[1])
    return [spec(2, 1, 2, 6.0, n=n + (1,), mu=mu, eps=eps, inc_dir=(np.cos(t), np.sin(t), 0.0),
                 inc_pol=(-np.sin(t), np.cos(t), 0.0)) for t in np.linspace(0.1, 1.2, count)]


CHILD = """
import sys, numpy as np, torch
torch.cuda.set_device(0)
import paper_2105_11993_amd as thm
from tests.test_gpu_cells_batches import members
count, out = int(sys.argv[1]), sys.argv[2]
Ss = [thm.thm_assemble(d) for d in members(count)]
i = Ss[0].info
cells = i["n_cells"]
skel = i["n_dofs"] - 12 * cells  # degree 2: 12 functions of a cell are interior, 12 are not
res = {}
for prec, w, kw in ((thm.THM_FP64, 8, dict(rtol=1e-13)), (thm.THM_FP32_IR, 4, dict(rtol=1e-11))):
    o = thm.default_opts(precision=prec, **kw)
    Es, st = thm.thm_gmres_solve(Ss, o, allow_not_converged=True)
    # again, every third system from its solution: it stops at once, the others go on beside it
    E0 = [E.clone() if k % 3 == 0 else torch.zeros_like(E) for k, E in enumerate(Es)]
    Fs, st = thm.thm_gmres_solve(Ss, o, E0, allow_not_converged=True)
    for k in range(count):
        res[f"e{prec}_{k}"], res[f"f{prec}_{k}"] = Es[k].cpu().numpy(), Fs[k].cpu().numpy()
    ms, by = thm.thm_time_spmv_systems(Ss, precision=prec, reps=1)
    want = cells * (8 * 12 + 8) + 4 * (skel + 1) + sum(
        4 * w * (S.n + 12 * cells) + (w + 4) * S.info["nnz_c"] + 4 * skel for S in Ss)
    assert by == want, (by, want)  # the bytes of code 30
    print("members", count, prec, [s["iters"] for s in st], flush=True)
np.savez(out, **res)
"""


@pytest.mark.parametrize("count", sorted(GROUPS))
def test_members_of_a_group(tmp_path, count):
    print("case cells, group of", count, flush=True)
    cache = tmp_path / "tune"
    cache.write_text("".join(f"gfx950:d2:p2:n{n}:b{count}:g1:{p}:cells 30\n" for n in range(8, 24)
                             for p in ("fp64", "fp32")))
    r = subprocess.run([sys.executable, "-c", CHILD, str(count), str(tmp_path / "out.npz")], cwd=ROOT,
                       capture_output=True, text=True, timeout=100, env=dict(os.environ, THM_TUNE_CACHE=str(cache)))
    print(r.stdout, r.stderr, flush=True)
    assert r.returncode == 0
    out = np.load(tmp_path / "out.npz")
    for k, d in enumerate(members(count)):
        if k not in (0, 1, 3, count // 2, count - 1):
            continue
        Eo = system.solve_lu(system.assemble(problem(d)))
        for prec, bar in ((0, 1e-10), (1, 1e-8)):  # the bars of tight solves in the two precisions
            for v in "ef":
                assert rel(out[f"{v}{prec}_{k}"], Eo) <= bar, (k, prec, v)


def test_several_rounds_of_tiles():
    import torch
    import paper_2105_11993_amd as thm
    print("case cells, rounds", flush=True)
    n = (517, 301, 1)  # 19,453 tiles of 8 cells: more than 2 x 8192 waves, the last one partly filled
    rng = np.random.default_rng(44)
    S = thm.thm_assemble(spec(2, 1, 0, 30.0, n=n, mu=rng.uniform(0.5, 2.0, n[0] * n[1])))
    (kr, kc, kv), (cr, cc, cv) = thm.thm_export_matrices(S)
    keep = sp.diags((thm.thm_export_rhs(S)[0] == 0).astype(float))
    A = sp.csr_matrix((kv, kc, kr), shape=(S.n, S.n)) + 1j * sp.csr_matrix((cv, cc, cr), shape=(S.n, S.n))
    A = keep @ A @ keep + (sp.identity(S.n) - keep)
    x = rng.standard_normal(S.n) + 1j * rng.standard_normal(S.n)
    for prec, eps in ((thm.THM_FP64, 2.0 ** -53), (thm.THM_FP32_IR, 2.0 ** -24)):
        thm.thm_set_spmv_variant(S, prec, thm.THM_SPMV_CELLS)
        y = thm.thm_apply_operator(S, torch.from_numpy(x).cuda(), precision=prec).cpu().numpy()
        # up to 4 products from each of 2 cells and 2 of C, both terms of an entry rounded: below 4 |K| row sums
        assert np.abs(y - A @ x).max() <= 4 * 20 * eps * (abs(A) @ abs(x)).max(), prec
