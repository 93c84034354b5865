"""The nested-dissection form of the factorised K^{-1} (the default) against the oracle, at the
shapes where its tree can go wrong: a root alone, strips, uneven boxes, boxes of one cell whose own
set is empty, four boxes around a 3D edge, fronts beyond one staged chunk, factor groups of one, two,
nine and seventeen members (vector units, one and two n tiles, a second member chunk), and a mesh close
to a resonance of its boxes, where FP32 solves take another tree.

Each test prints its case before touching the GPU.
"""
import numpy as np
import pytest

from oracle import system
from tests._gpu_helpers import dirichletized, problem, rel, spec

pytestmark = pytest.mark.gpu


def box(dim, n, p, omega, **kw):
    return spec(dim, 1, p, omega, **dict(kw, n=tuple(n) + (1,) * (3 - dim)))


CASES = [box(2, (1, 9), 1, 5.0), box(2, (37, 2), 0, 6.0), box(2, (5, 3), 3, 4.0), box(2, (23, 18), 2, 9.0),
         box(2, (70, 66), 0, 11.0), box(3, (1, 1, 7), 1, 3.0), box(3, (5, 4, 6), 1, 5.0), box(3, (7, 9, 3), 0, 4.0)]


def _ids(c):
    return f"d{c['dim']}n{'x'.join(str(v) for v in c['n'][:c['dim']])}p{c['p']}"


@pytest.fixture(scope="module")
def thm():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2105_11993_amd as t
    return t


@pytest.mark.parametrize("d", CASES, ids=_ids)
def test_inverts_k(thm, d):
    import torch
    rng = np.random.default_rng(91)
    d = dict(d, mu=rng.uniform(1.0, 2.0, int(np.prod(d["n"]))))
    print("case nd", _ids(d), flush=True)
    S = thm.thm_assemble(d)
    K = dirichletized(system.assemble(problem(d)))[0].real
    x = rng.standard_normal(S.n) + 1j * rng.standard_normal(S.n)
    xt = torch.from_numpy(x).cuda()
    knorm = abs(K).sum(axis=1).max()

    def eta(z):  # normwise backward error; the bars of the other factor forms
        return np.linalg.norm(K @ z - x, np.inf) / (knorm * np.linalg.norm(z, np.inf) + np.linalg.norm(x, np.inf))

    for prec, bar in ((thm.THM_FP64, 1e-11), (thm.THM_FP32_IR, 1e-4)):
        z = thm.thm_apply_precond(S, xt, precision=prec)
        assert eta(z.cpu().numpy()) <= bar, prec
        y = torch.full_like(xt, complex(float("nan"), float("nan")))
        thm.thm_apply_precond_noalloc(S, xt, y, precision=prec)
        torch.cuda.synchronize()
        assert np.array_equal(y.cpu().numpy(), z.cpu().numpy())


@pytest.mark.parametrize("count", [2, 9, 17])
@pytest.mark.parametrize("mixed", [False, True], ids=["fp64", "mixed"])
def test_groups_of_systems_with_one_factor(thm, count, mixed):
    """Systems that share K (same mesh, other incidence) are the columns of one apply."""
    print("case nd group", count, mixed, flush=True)
    specs = []
    for i in range(count):
        th = 0.1 + 0.05 * i
        specs.append(box(2, (21, 14), 2, 7.0, inc_dir=(np.cos(th), np.sin(th), 0.0),
                         inc_pol=(-np.sin(th), np.cos(th), 0.0)))
    systems = [thm.thm_assemble(d) for d in specs]
    o = thm.default_opts(rtol=1e-11, precision=thm.THM_FP32_IR) if mixed else thm.default_opts(rtol=1e-13)
    Es, sts = thm.thm_gmres_solve(systems, o)
    for d, E in zip(specs, Es):
        assert rel(E.cpu().numpy(), system.solve_lu(system.assemble(problem(d)))) <= (1e-8 if mixed else 1e-10)


def test_fp32_solve_close_to_a_resonance_of_the_boxes(thm):
    """w L = 6.25 on 32^2 cells: boxes of a quarter of the side resonate within 1%, the FP32 form of the
    default tree has a residual of 1e-3 there.  A refinement step has to gain three digits or more, as it
    does away from the resonance, so four steps reach 1e-11."""
    d = box(2, (32, 32), 1, 6.25)
    print("case nd resonance", flush=True)
    S = thm.thm_assemble(d)
    (E,), (st,) = thm.thm_gmres_solve([S], thm.default_opts(rtol=1e-11, restart=80, precision=thm.THM_FP32_IR))
    assert st["refinements"] <= 4 and st["gmres_ir"] == 0, st
    assert rel(E.cpu().numpy(), system.solve_lu(system.assemble(problem(d)))) <= 1e-8
