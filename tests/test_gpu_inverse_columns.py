"""Blocked inversion of a matrix of more than 16,384 rows, whose strips are single columns in memory: the
inner matrix of the complete inverse on a strip of 2 x 4101 cells with open long sides.
"""
import numpy as np
import pytest

from oracle import system
from tests._gpu_helpers import dirichletized, problem, spec

pytestmark = pytest.mark.gpu


def test_complete_inverse_of_a_long_strip():
    import torch
    import paper_2105_11993_amd as thm
    n = (2, 4101, 1)
    rng = np.random.default_rng(9)
    d = spec(2, 1, 0, 3.0, n=n, hi=(0.2, 410.1, 1.0), inc_faces=4, inc_dir=(0.0, 1.0, 0.0), inc_pol=(1.0, 0.0, 0.0),
             mu=rng.uniform(1.0, 2.0, 2 * 4101))
    A = dirichletized(system.assemble(problem(d)))[0]
    size = 2 * int((abs(A.imag).sum(axis=1) > 0).sum())
    print("case inverse by columns", size, flush=True)
    assert 16384 < size < 16500
    S = thm.thm_assemble(d)
    x = rng.standard_normal(S.n) + 1j * rng.standard_normal(S.n)
    z = thm.thm_apply_precond_full(S, torch.from_numpy(x).cuda()).cpu().numpy()
    an = abs(A).sum(axis=1).max()
    eta = np.linalg.norm(A @ z - x, np.inf) / (an * np.linalg.norm(z, np.inf) + np.linalg.norm(x, np.inf))
    print("  ", eta, flush=True)
    assert eta <= 1e-11  # the bar of the exact factor forms
