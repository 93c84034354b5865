"""Wide fronts of factor groups: the matrix-core products read their operands without a stage, eight waves
share a front of more than 384 columns, and the root has no boundary behind its padded columns.  Groups
of 1, 2, 8, 9 and 17 members (vector units; one and two tiles of members; a second chunk) against the
oracle, in both precisions.
"""
import numpy as np
import pytest

from oracle import system
from tests._gpu_helpers import FP64_TIGHT, MIXED_TIGHT, problem, rel, spec

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def thm():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2105_11993_amd as t
    return t


@pytest.mark.parametrize("mixed", [False, True], ids=["fp64", "mixed"])
@pytest.mark.parametrize("count", [1, 2, 8, 9, 17])
@pytest.mark.parametrize("dim,n,p", [(3, (4, 5, 5), 1), (2, (33, 29), 2)], ids=["3d", "2d"])
def test_groups_with_wide_fronts(thm, dim, n, p, count, mixed):
    rng = np.random.default_rng(31)
    mu = rng.uniform(1.0, 2.0, int(np.prod(n)))
    print("case wide fronts", n, count, mixed, flush=True)
    ds = []
    for t in np.linspace(0.1, 1.2, count):
        c, s = np.cos(t), np.sin(t)
        ds.append(spec(dim, 1, p, 5.0, n=tuple(n) + (1,) * (3 - dim), mu=mu, inc_dir=(c, s, 0.0), inc_pol=(-s, c, 0.0)))
    Ss = [thm.thm_assemble(d) for d in ds]
    kw = dict(MIXED_TIGHT, precision=thm.THM_FP32_IR) if mixed else FP64_TIGHT
    Es, st = thm.thm_gmres_solve(Ss, thm.default_opts(**kw), allow_not_converged=True)
    for d, E in list(zip(ds, Es))[:: max(1, count - 1)]:
        assert rel(E.cpu().numpy(), system.solve_lu(system.assemble(problem(d)))) <= (1e-8 if mixed else 1e-10)
