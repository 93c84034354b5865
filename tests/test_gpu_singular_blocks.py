"""Blocks that are exactly singular while K is factorised.

Cells of side 2^27 whose mu is near the largest double and whose eps is the smallest have an element matrix
of zeros: their interior block K_ii is singular, which every form of the factor reports.  Boxes of the
nested dissection may be singular where K is not; another tree is taken then.
"""
import numpy as np
import pytest
import scipy.sparse as sp

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


def singular_pair(thm):
    """eps (with mu = 3) of a cell of degree 0 whose matrix is exactly singular on its upper and left edge:
    w^2 eps M = 2 curl / 3 to the last bit, so the block is -curl / 3 [[1, -1], [-1, 1]]."""
    tries = 2.0 * UNIT * (1.0 + np.arange(-32, 32) * 2.0 ** -52)
    S = thm.thm_assemble(huge(8, 0, np.full(64, 3.0), tries))
    for eps, e in zip(tries, thm.thm_export_elements(S, 0, 64, 4)):
        b = e[np.ix_([1, 2], [1, 2])]
        if b[0, 0] == b[1, 1] and b[0, 1] == b[1, 0] and abs(b[0, 1]) == abs(b[0, 0]):
            return eps
    raise AssertionError("no such cell")


def test_boxes_singular_at_some_levels(thm):
    """16^2 cells of degree 0 are halved into boxes of 4 x 8, 4 x 4, 2 x 4 and 2 x 2 cells, and the tree that
    costs least starts at those of 4 x 4.  A cell of the special kind in the lower right corner of such a box,
    next to two cells of zeros, leaves its two inner edges without other neighbours: the boxes of 4 x 4
    cells and less that hold it are exactly singular, those of 4 x 8 and K itself are not."""
    import torch
    print("case singular boxes", flush=True)
    rng = np.random.default_rng(13)
    n = 16
    mu, eps = rng.uniform(1.0, 2.0, (n, n)), rng.uniform(0.6, 0.9, (n, n)) * UNIT
    mu[4, 7], eps[4, 7] = 3.0, singular_pair(thm)
    for j, i in ((4, 6), (5, 7)):
        mu[j, i], eps[j, i] = NO_MU, NO_EPS
    S = thm.thm_assemble(huge(n, 0, mu.ravel(), eps.ravel()))
    (kr, kc, kv), _ = thm.thm_export_matrices(S)
    free = thm.thm_export_rhs(S)[0] == 0
    K = sp.csr_matrix((kv, kc, kr), shape=(S.n, S.n)).toarray()
    K[~free, :] = 0.0
    K[:, ~free] = 0.0
    K[~free, ~free] = 1.0
    x = rng.standard_normal(S.n) + 1j * rng.standard_normal(S.n)
    x[~free] = 0.0
    for prec, bar in ((thm.THM_FP64, 1e-11), (thm.THM_FP32_IR, 1e-4)):  # the bars of the factor forms
        z = thm.thm_apply_precond(S, torch.from_numpy(x).cuda(), precision=prec).cpu().numpy()
        Kf = K[np.ix_(free, free)]
        r = np.linalg.norm(Kf @ z[free] - x[free], np.inf)
        eta = r / (abs(Kf).sum(axis=1).max() * np.linalg.norm(z, np.inf) + np.linalg.norm(x, np.inf))
        print("  ", prec, eta, flush=True)
        assert eta <= bar
