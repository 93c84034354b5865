"""The first step x += (K + iC)^{-1} (b - (K + iC) x) of FP64 solves with the complete inverse: from zero and
from a guess, ended by the iteration limit, by a loose tolerance and by one that no step reaches (where
steps that do not reduce the residual are undone), with systems of a batch that need different numbers
of steps, and in a decomposition with and without captured graphs.
"""
import numpy as np
import pytest

from oracle import system
from tests._gpu_helpers import dirichletized, problem, rel, spec

pytestmark = pytest.mark.gpu


def box(dim, n, p, **kw):
    return spec(dim, 1, p, 5.0, **dict(kw, n=tuple(n) + (1,) * (3 - dim)))


@pytest.fixture(scope="module")
def thm():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2105_11993_amd as t
    return t


@pytest.mark.parametrize("d", [box(2, (1, 1), 0), box(2, (13, 6), 2), box(3, (4, 3, 5), 1)], ids=["1cell", "2d", "3d"])
def test_guesses_limits_and_tolerances(thm, d):
    import torch
    print("case first step", d["n"], flush=True)
    S = thm.thm_assemble(d)
    Eo = system.solve_lu(system.assemble(problem(d)))
    D = dirichletized(system.assemble(problem(d)))[1]
    rng = np.random.default_rng(3)

    def run(E0, **kw):
        E = torch.from_numpy(E0.copy()).cuda()
        out, st = thm.thm_gmres_solve(S, thm.default_opts(precond=thm.THM_PREC_FULL, **kw), [E], allow_not_converged=True)
        return out[0].cpu().numpy(), st[0]

    zero = np.zeros(S.n, complex)
    guess = Eo + rng.standard_normal(S.n) * (~D)
    for E0 in (zero, guess):
        E, st = run(E0, rtol=1e-10)
        assert st["status"] == 0 and st["iters"] <= 2 and rel(E, Eo) <= 1e-9
        E, st = run(E0, rtol=1e-2)
        assert st["status"] == 0 and st["iters"] == 1 and rel(E, Eo) <= 1e-8
        E, st = run(E0, rtol=1e-10, max_iter=0)
        assert st["iters"] == 0 and np.array_equal(E[~D], E0[~D])
        # no step reaches this tolerance, and none may make a solved system worse
        E, st = run(E0, rtol=1e-30, max_iter=6)
        assert st["iters"] <= 6 and rel(E, Eo) <= 1e-10
    E, st = run(Eo, rtol=1e-30, max_iter=4)
    assert rel(E, Eo) <= 1e-10


def test_batch_of_systems_at_different_residuals(thm):
    import torch
    print("case first step, batch", flush=True)
    ds = [box(2, (6, 5), 1), box(2, (9, 4), 2), box(3, (2, 3, 2), 1)]
    Ss = [thm.thm_assemble(d) for d in ds]
    Eo = [system.solve_lu(system.assemble(problem(d))) for d in ds]
    E0 = [np.zeros(Ss[0].n, complex), Eo[1], np.zeros(Ss[2].n, complex)]
    o = thm.default_opts(precond=thm.THM_PREC_FULL, rtol=1e-9)
    Es, st = thm.thm_gmres_solve(Ss, o, [torch.from_numpy(e.copy()).cuda() for e in E0])
    assert st[1]["iters"] == 0 and 1 <= st[0]["iters"] <= 2 and 1 <= st[2]["iters"] <= 2
    for E, e in zip(Es, Eo):
        assert rel(E.cpu().numpy(), e) <= 1e-8


@pytest.mark.parametrize("kw", [{}, {"use_graph": 0}, {"batched": 0}, {"relax_inner": 0}],
                         ids=["default", "no_graph", "sequential", "tight"])
def test_decomposition(thm, kw):
    print("case first step, decomposition", kw, flush=True)
    d = spec(2, 8, 1, 5.0, subdomains=(2, 2, 1), mu=np.random.default_rng(4).uniform(1.0, 2.0, 64))
    S = thm.thm_assemble(d)
    o = thm.default_opts(precond=thm.THM_PREC_FULL, rtol=1e-11, inner_rtol=1e-13, ddm_outer=thm.THM_DDM_GMRES, **kw)
    E, st = thm.thm_ddm_solve(S, o)
    assert st["rel_residual"] <= 1e-11
    assert rel(E.cpu().numpy(), system.solve_lu(system.assemble(problem(d)))) <= 1e-9
