"""Blocked inversion of dense blocks, through the complete inverse of K + iC: its inner matrix has two
rows per boundary DoF with C, so the mesh sets the size and with it the rows that a thread of the
strip kernel holds (1, 2, up to 4, 8, 16 and 32 of 512).  Sizes are no multiples of a strip, a panel
or a block of 512; the last case inverts several blocks of different sizes at once.
"""
import numpy as np
import pytest

from oracle import system
from tests._gpu_helpers import dirichletized, problem, spec

pytestmark = pytest.mark.gpu


def box(dim, n, p):
    return spec(dim, 1, p, 4.0, n=tuple(n) + (1,) * (3 - dim))


# mesh, and the rows a thread holds
CASES = [(box(2, (9, 7), 1), 1), (box(2, (60, 50), 2), 2), (box(3, (4, 4, 4), 1), 3), (box(3, (6, 7, 6), 1), 7),
         (box(3, (10, 10, 9), 1), 15), (box(3, (11, 11, 11), 1), 19)]


def eta(A, z, x):  # normwise backward error
    an = abs(A).sum(axis=1).max()
    return np.linalg.norm(A @ z - x, np.inf) / (an * np.linalg.norm(z, np.inf) + np.linalg.norm(x, np.inf))


@pytest.mark.parametrize("d,rows", CASES, ids=[str(c[1]) for c in CASES])
def test_complete_inverse_at_every_strip_form(d, rows):
    import torch
    import paper_2105_11993_amd as thm
    rng = np.random.default_rng(7)
    d = dict(d, mu=rng.uniform(1.0, 2.0, int(np.prod(d["n"]))))
    A = dirichletized(system.assemble(problem(d)))[0]
    size = 2 * int((abs(A.imag).sum(axis=1) > 0).sum())
    print("case inverse", d["n"], size, flush=True)
    assert -(-size // 512) == rows
    S = thm.thm_assemble(d)
    x = rng.standard_normal(S.n) + 1j * rng.standard_normal(S.n)
    z = thm.thm_apply_precond_full(S, torch.from_numpy(x).cuda()).cpu().numpy()
    assert eta(A, z, x) <= 1e-11  # the bar of the exact factor forms


def test_blocks_of_different_sizes_together():
    import torch
    import paper_2105_11993_amd as thm
    rng = np.random.default_rng(8)
    ds = [dict(box(2, n, p), mu=rng.uniform(1.0, 2.0, n[0] * n[1]))
          for n, p in (((4, 4), 0), ((17, 9), 1), ((23, 31), 2), ((40, 12), 1))]
    print("case inverses of different sizes", flush=True)
    Ss = [thm.thm_assemble(d) for d in ds]
    Es, st = thm.thm_gmres_solve(Ss, thm.default_opts(rtol=1e-12, precond=thm.THM_PREC_FULL))
    for d, E, s in zip(ds, Es, st):
        Eo = system.solve_lu(system.assemble(problem(d)))
        assert s["rel_residual"] <= 1e-12
        assert np.linalg.norm(E.cpu().numpy() - Eo) <= 1e-9 * np.linalg.norm(Eo)
    torch.cuda.synchronize()
