"""Device memory over many changes of mu: what a solve keeps for one mu is given back with the next."""
import numpy as np
import pytest

from tests._gpu_helpers import spec

pytestmark = pytest.mark.gpu

MIB = float(1 << 20)


def free_mib():
    import torch
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0] / MIB


@pytest.fixture(scope="module")
def thm():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2105_11993_amd as t
    return t


def test_repeated_changes_of_mu(thm):
    """Every change drops the system's context with its stream, about 1 MiB of device memory each."""
    import torch
    print("case memory, same mu", flush=True)
    S = thm.thm_assemble(spec(2, 16, 1, 6.0))
    mu = torch.ones(256, dtype=torch.float64, device="cuda")

    def steps(count):
        for _ in range(count):
            thm.thm_system_set_mu(S, mu)
            thm.thm_gmres_solve([S], thm.default_opts(rtol=1e-6))
        return free_mib()

    before = steps(10)
    after = steps(60)
    print("  ", before, after, flush=True)
    assert before - after < 16.0


def test_plans_kept_by_systems_of_one_mesh(thm):
    """mu scans resonances of the boxes, so that solves choose ever other trees; a system keeps eight plans, also
    of those that another system of its batch built first."""
    import torch
    print("case memory, plans", flush=True)
    n = 96
    Ss = [thm.thm_assemble(spec(2, n, 1, 15.0, mu=np.full(n * n, v))) for v in (1.0, 1.01)]
    rng = np.random.default_rng(1)

    def step(*mus):
        for S, v in zip(Ss, mus):
            thm.thm_system_set_mu(S, torch.full((n * n,), v, dtype=torch.float64, device="cuda"))
        thm.thm_gmres_solve(Ss, thm.default_opts(max_iter=1, rtol=1e-2), allow_not_converged=True)
        for S in Ss:
            thm.thm_system_release_workspaces(S)

    def scan(count):
        for _ in range(count):
            step(*rng.uniform(0.2, 10.0, 2))
        step(1.0, 1.01)  # factors of the same size each time
        return free_mib()

    before = scan(30)
    after = scan(60)
    print("  ", before, after, flush=True)
    assert before - after < 16.0  # a plan here takes up to 2 MiB
