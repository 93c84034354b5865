"""A mesh whose factorisation is refused is refused again by the next call: the first leaves no half-made
factor behind."""
import pytest

from tests._gpu_helpers import spec

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", ["", "bcr", "lu"])
def test_refused_twice(monkeypatch, form):
    import torch
    import paper_2105_11993_amd as thm
    print("case refused factor", form, flush=True)
    monkeypatch.setenv("THM_FACTOR_FORM", form) if form else monkeypatch.delenv("THM_FACTOR_FORM", raising=False)
    S = thm.thm_assemble(spec(2, 1, 1, 5.0, n=(20000, 1, 1)))  # two layers of 80,000 and 40,000 DoFs
    x = torch.ones(S.n, dtype=torch.complex128, device="cuda")
    for _ in range(2):
        for call in (lambda: thm.thm_apply_precond(S, x), lambda: thm.thm_gmres_solve(S, thm.default_opts(max_iter=1)),
                     lambda: thm.thm_apply_precond_noalloc(S, x, torch.empty_like(x))):
            with pytest.raises(thm.ThmError):
                call()
    assert S.fresh_info()["factor_bytes"] == -1
