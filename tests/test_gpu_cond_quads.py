"""Interior recovery of four systems at a time: batches large enough for it (1024 blocks), with a last
quad of three and of one member, two factors, and some systems that converge before the others, against
solves of one system each.
"""
import numpy as np
import pytest

from tests._gpu_helpers import rel, spec

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def thm():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2105_11993_amd as t
    return t


@pytest.mark.parametrize("mixed", [False, True], ids=["fp64", "mixed"])
@pytest.mark.parametrize("counts", [(15,), (17,), (9, 8)], ids=["15", "17", "two_factors"])
def test_large_groups_equal_single_solves(thm, counts, mixed):
    import torch
    rng = np.random.default_rng(12)
    print("case quads", counts, mixed, flush=True)
    Ss = []
    for count in counts:
        mu = rng.uniform(1.0, 2.0, 64 * 64)
        for t in np.linspace(0.1, 1.2, count):
            c, s = np.cos(t), np.sin(t)
            Ss.append(thm.thm_assemble(spec(2, 64, 2, 6.0, mu=mu, inc_dir=(c, s, 0.0), inc_pol=(-s, c, 0.0))))
    o = thm.default_opts(rtol=1e-11, precision=thm.THM_FP32_IR if mixed else thm.THM_FP64)
    one = thm.default_opts(rtol=1e-11, batched=0)
    ref, _ = thm.thm_gmres_solve(Ss, one)
    # every third system starts from its solution and stops at once
    E0 = [e.clone() if i % 3 == 1 else torch.zeros_like(e) for i, e in enumerate(ref)]
    Es, st = thm.thm_gmres_solve(Ss, o, E0)
    for i, (E, e) in enumerate(zip(Es, ref)):
        assert rel(E.cpu().numpy(), e.cpu().numpy()) <= 1e-8, i  # two solves to 1e-11
