"""Blocks that are exactly singular while K is factorised.

Cells of side 2^27 whose mu is near the largest double and whose eps is the smallest have an element matrix
of zeros: their interior block K_ii is singular, which every form of the factor reports.
"""
import numpy as np
import pytest

from tests._gpu_helpers import spec

pytestmark = pytest.mark.gpu

H = 2.0 ** 27  # the curl term of a cell is of the order of 1 / H^2 = 2^-54, the mass term of order w^2 eps
UNIT = 2.0 ** -54
NO_MU, NO_EPS = 1.7e308, 5e-324  # 1 / mu / H^2 and w^2 eps / 3 round to zero


def huge(n, p, mu, eps, **kw):
    return spec(2, 1, p, 1.0, **dict(kw, n=(n, n, 1), hi=(n * H, n * H, 1.0), mu=mu, eps=eps))


@pytest.fixture(scope="module")
def thm():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2105_11993_amd as t
    return t


@pytest.mark.parametrize("form", ["", "bcr", "lu"])
@pytest.mark.parametrize("n", [3, 16], ids=["root_alone", "tree"])
def test_singular_interior_block_is_reported(thm, monkeypatch, n, form):
    import torch
    print("case singular interior", n, form, flush=True)
    monkeypatch.setenv("THM_FACTOR_FORM", form) if form else monkeypatch.delenv("THM_FACTOR_FORM", raising=False)
    rng = np.random.default_rng(12)
    mu, eps = rng.uniform(1.0, 2.0, n * n), rng.uniform(0.1, 0.3, n * n) * UNIT
    cell = (n // 2) * n + n // 2
    mu[cell], eps[cell] = NO_MU, NO_EPS
    S = thm.thm_assemble(huge(n, 1, mu, eps))
    assert not thm.thm_export_elements(S, cell, 1, 12).any()
    x = torch.ones(S.n, dtype=torch.complex128, device="cuda")
    for call in (lambda: thm.thm_apply_precond(S, x), lambda: thm.thm_apply_precond(S, x, precision=thm.THM_FP32_IR),
                 lambda: thm.thm_gmres_solve(S, thm.default_opts(max_iter=2), allow_not_converged=True)):
        with pytest.raises(thm.ThmError) as e:
            call()
        assert e.value.code == -5
