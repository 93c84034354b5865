"""First steps of FP64 solves with the complete inverse that do harm, and systems that take none."""
import numpy as np
import pytest

from oracle import system
from tests._gpu_helpers import dirichletized, problem, spec

pytestmark = pytest.mark.gpu


def box(dim, n, p, **kw):
    return spec(dim, 1, p, 5.0, **dict(kw, n=tuple(n) + (1,) * (3 - dim)))


@pytest.fixture(scope="module")
def thm():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2105_11993_amd as t
    return t


def test_solved_system_beside_one_that_is_finished_in_fp64(thm):
    """A system whose guess meets the tolerance takes no step in a mixed solve that ends with FP64 steps of
    the other (no refinement, two steps of GMRES-based refinement allowed), for which the tolerance is
    out of reach.  The solves before this one left a step and then residuals that are not numbers in the
    workspace."""
    import torch
    print("case first step beside a solved system", flush=True)
    ds = [box(2, (1, 1), 0), box(2, (13, 6), 2)]
    Ss = [thm.thm_assemble(d) for d in ds]
    Eo = [system.solve_lu(system.assemble(problem(d))) for d in ds]
    opts = dict(precond=thm.THM_PREC_FULL, rtol=3e-16, restart=1, max_iter=2)
    (E,), (st,) = thm.thm_gmres_solve(Ss[0], thm.default_opts(**dict(opts, max_iter=6)))
    guess0 = E.clone()
    for v in (1.0, float("nan")):
        guess = [torch.full((S.n,), complex(v, 0.0), dtype=torch.complex128, device="cuda") for S in Ss]
        thm.thm_gmres_solve(Ss, thm.default_opts(**opts), guess, allow_not_converged=True)
    E0 = [guess0.clone(), torch.zeros(Ss[1].n, dtype=torch.complex128, device="cuda")]
    Es, st = thm.thm_gmres_solve(Ss, thm.default_opts(precision=thm.THM_FP32_IR, max_refine=0, **opts), E0,
                                 allow_not_converged=True)
    print("  ", st, flush=True)
    assert st[1]["fp64_fallback"] == 1 and st[0]["fp64_fallback"] == 0 and st[0]["status"] == 0
    assert torch.equal(Es[0], guess0)
    assert np.linalg.norm(Es[1].cpu().numpy() - Eo[1]) <= 1e-9 * np.linalg.norm(Eo[1])


def test_iteration_limit_of_one(thm):
    """From a guess at rounding level the first step may end further off; the limit is reached after it, and
    the better of the two vectors is returned."""
    import torch
    print("case first step, limit of one", flush=True)
    rng = np.random.default_rng(21)
    for k in range(24):
        d = box(2, (4 + k % 5, 3 + k % 7), k % 3, mu=rng.uniform(1.0, 2.0, (4 + k % 5) * (3 + k % 7)))
        S = thm.thm_assemble(d)

        def run(E, max_iter):
            o = thm.default_opts(precond=thm.THM_PREC_FULL, rtol=1e-30, max_iter=max_iter)
            (E,), (st,) = thm.thm_gmres_solve(S, o, [E.clone()], allow_not_converged=True)
            return E, st["rel_residual"], st["iters"]

        E0, before, _ = run(torch.from_numpy(system.solve_lu(system.assemble(problem(d)))).cuda(), 6)
        E0, before, n0 = run(E0, 0)
        E1, after, n1 = run(E0, 1)
        assert n0 == 0 and n1 <= 1 and after <= before, (k, before, after)


def test_step_that_is_not_finite(thm):
    """Cells of side 2^500: K is of the order of 2^-1000 and C of 2^-500, so the first step from a guess of the
    order of 2^1000 overflows, while the residual does not.  At the iteration limit the guess is returned."""
    import torch
    print("case first step, not finite", flush=True)
    h = 2.0 ** 500
    rng = np.random.default_rng(22)
    d = spec(2, 1, 0, 1.0, n=(5, 4, 1), hi=(5 * h, 4 * h, 1.0), mu=rng.uniform(1.0, 2.0, 20),
            eps=rng.uniform(0.1, 0.3, 20) * 2.0 ** -1000)
    S = thm.thm_assemble(d)
    free = thm.thm_export_rhs(S)[0] == 0
    E0 = (rng.standard_normal(S.n) + 1j * rng.standard_normal(S.n)) * 2.0 ** 1000 * free
    o = thm.default_opts(precond=thm.THM_PREC_FULL, rtol=1e-10, max_iter=1)
    (E,), (st,) = thm.thm_gmres_solve(S, o, [torch.from_numpy(E0.copy()).cuda()], allow_not_converged=True)
    print("  ", st, flush=True)
    assert st["iters"] == 1 and np.isfinite(st["rel_residual"])
    assert np.array_equal(E.cpu().numpy()[free], E0[free])
