"""The product from the cells' reference matrices (SpMV code 30) against the product with the oracle's
assembled matrix and against code 19: every element, material in both terms, Dirichlet rows, both
signs of C, fewer than the 8 cells of a tile, the last tile of a block, more cells than one round of
blocks, groups of 1, 2, 9 and 16 members with different vectors, and K that the cells do not hold.
"""
import numpy as np
import pytest

from oracle import system
from tests._gpu_helpers import FP64_TIGHT, dirichletized, problem, rel, spec

pytestmark = pytest.mark.gpu


def box(dim, n, p, **kw):
    return spec(dim, 1, p, 5.0, **dict(kw, n=tuple(n) + (1,) * (3 - dim)))


CASES = [box(2, (1, 1), 0), box(2, (1, 7), 3), box(2, (9, 5), 0), box(2, (33, 4), 1), box(2, (11, 13), 2, inc_faces=5),
         box(2, (8, 8), 3), box(3, (1, 1, 1), 1), box(3, (3, 5, 2), 0), box(3, (4, 3, 5), 1, inc_faces=18)]


@pytest.fixture(scope="module")
def thm():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2105_11993_amd as t
    return t


@pytest.mark.parametrize("d", CASES, ids=[f"{'x'.join(map(str, c['n'][:c['dim']]))}p{c['p']}" for c in CASES])
def test_product_matches_the_assembled_matrix(thm, d):
    import torch
    rng = np.random.default_rng(5)
    nc = int(np.prod(d["n"]))
    d = dict(d, mu=rng.uniform(0.5, 2.0, nc), eps=rng.uniform(1.0, 3.0, nc))
    print("case cells", d["n"], d["p"], flush=True)
    S = thm.thm_assemble(d)
    A = dirichletized(system.assemble(problem(d)))[0]
    x = rng.standard_normal(S.n) + 1j * rng.standard_normal(S.n)
    xt = torch.from_numpy(x).cuda()
    for prec, eps in ((thm.THM_FP64, 2.0 ** -53), (thm.THM_FP32_IR, 2.0 ** -24)):
        thm.thm_set_spmv_variant(S, prec, thm.THM_SPMV_CELLS)
        for tr in (False, True):
            y = thm.thm_apply_operator(S, xt, transpose=tr, precision=prec).cpu().numpy()
            B = A.conj() if tr else A
            # both terms of an entry are rounded: |curl| / mu + w^2 eps |mass| is below 4 |K| row sums here,
            # and a row adds up to 54 products from each of up to 4 cells
            bar = 4 * 220 * eps * (abs(B) @ abs(x)).max()
            assert np.abs(y - B @ x).max() <= bar, (prec, tr)


@pytest.mark.parametrize("count", [1, 2, 9, 16])
def test_members_of_a_group(thm, count):
    import torch
    rng = np.random.default_rng(6)
    mu = rng.uniform(1.0, 2.0, 70)
    print("case cells, members", count, flush=True)
    ds = [box(2, (10, 7), 1, mu=mu, inc_dir=(np.cos(t), np.sin(t), 0.0), inc_pol=(-np.sin(t), np.cos(t), 0.0))
          for t in np.linspace(0.1, 1.2, count)]
    Ss = [thm.thm_assemble(d) for d in ds]
    Es, st = thm.thm_gmres_solve(Ss, thm.default_opts(**FP64_TIGHT), allow_not_converged=True)
    for d, E in zip(ds, Es):
        assert rel(E.cpu().numpy(), system.solve_lu(system.assemble(problem(d)))) <= 1e-10


@pytest.mark.parametrize("mixed", [False, True], ids=["fp64", "mixed"])
def test_subdomain_solves_with_the_product(thm, mixed):
    d = spec(2, 12, 2, 8.0, subdomains=(4, 4, 1), inc_dir=(np.cos(0.3), np.sin(0.3), 0.0),
             inc_pol=(-np.sin(0.3), np.cos(0.3), 0.0))
    print("case cells in a decomposition", mixed, flush=True)
    S = thm.thm_assemble(d)
    kw = dict(precision=thm.THM_FP32_IR) if mixed else {}
    o = thm.default_opts(**dict(FP64_TIGHT, rtol=1e-12, **kw))
    thm.thm_ddm_solve(S, o, allow_not_converged=True)
    for prec in (thm.THM_FP64, thm.THM_FP32_IR):
        thm.thm_set_spmv_variant(S, prec, thm.THM_SPMV_CELLS)
    E, st = thm.thm_ddm_solve(S, o, allow_not_converged=True)
    assert S.fresh_info()["ddm_spmv_variant"] == thm.THM_SPMV_CELLS
    Eo = system.solve_lu(system.assemble(problem(d)))
    print("  ", st, rel(E.cpu().numpy(), Eo), flush=True)
    assert rel(E.cpu().numpy(), Eo) <= 1e-10


def test_interface_terms_in_k_are_left_to_the_assembled_forms(thm):
    d = spec(2, 8, 1, 6.0, subdomains=(2, 2, 1), transmission=0.8 + 0.3j)
    print("case cells refused", flush=True)
    S = thm.thm_assemble(d)
    o = thm.default_opts(rtol=1e-10, inner_rtol=1e-12)
    E, st = thm.thm_ddm_solve(S, o, allow_not_converged=True)
    assert S.fresh_info()["ddm_spmv_variant"] != thm.THM_SPMV_CELLS
    with pytest.raises(thm.ThmError):
        thm.thm_set_spmv_variant(S, thm.THM_FP64, thm.THM_SPMV_CELLS)
    assert rel(E.cpu().numpy(), system.solve_lu(system.assemble(problem(d)))) <= 1e-8
