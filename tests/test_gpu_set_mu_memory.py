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
