"""Kernel-level calls on the caller's own vectors: in place, overlapping by all but one entry,
aligned to 8 bytes only, on another stream, and with nothing written beyond the vector.  The same
kernels run on the same values, so every result equals the plain call's bit by bit.
"""
import ctypes

import numpy as np
import pytest

from tests._gpu_helpers import spec

pytestmark = pytest.mark.gpu

# first 8-byte word of x and of y in one buffer of 4 n + 64 words (2 n words a vector)
LAYOUTS = {"apart": lambda n: (0, 2 * n + 8), "in_place": lambda n: (0, 0), "y_behind_x": lambda n: (0, 2),
           "y_before_x": lambda n: (2, 0), "adjacent": lambda n: (0, 2 * n), "x_misaligned": lambda n: (1, 2 * n + 8),
           "y_misaligned": lambda n: (0, 2 * n + 9)}


@pytest.mark.parametrize("precision", ["THM_FP64", "THM_FP32_IR"])
@pytest.mark.parametrize("d", [spec(2, 1, 0, 3.0), spec(2, 9, 2, 7.0), spec(3, 4, 1, 4.0)], ids=["1cell", "2d", "3d"])
def test_layouts_give_the_plain_result(d, precision):
    import torch
    import paper_2105_11993_amd as thm
    prec = getattr(thm, precision)
    print("case vectors", d["n"], precision, flush=True)
    S = thm.thm_assemble(d)
    rng = np.random.default_rng(17)
    x = torch.from_numpy(rng.standard_normal(S.n) + 1j * rng.standard_normal(S.n)).cuda()
    words = torch.view_as_real(x).reshape(-1)
    calls = {"operator": (thm.thm_apply_operator(S, x, precision=prec),
                          lambda xp, yp, st: thm._lib.thm_apply_operator(S.handle, 0, prec, xp, yp, st)),
             "precond": (thm.thm_apply_precond(S, x, precision=prec),
                         lambda xp, yp, st: thm._lib.thm_apply_precond(S.handle, prec, xp, yp, st))}
    streams = [torch.cuda.current_stream(), torch.cuda.Stream()]
    for name, (ref, call) in calls.items():
        ref = torch.view_as_real(ref).reshape(-1)
        for layout, at in LAYOUTS.items():
            for st in streams:
                with torch.cuda.stream(st):
                    xo, yo = at(S.n)
                    buf = torch.full((4 * S.n + 64,), 7.25, dtype=torch.float64, device="cuda")
                    buf[xo:xo + 2 * S.n] = words
                    rc = call(ctypes.c_void_p(buf.data_ptr() + 8 * xo), ctypes.c_void_p(buf.data_ptr() + 8 * yo),
                              ctypes.c_void_p(st.cuda_stream))
                    assert rc == 0, (name, layout)
                    assert torch.equal(buf[yo:yo + 2 * S.n], ref), (name, layout)
                    assert bool((buf[max(xo, yo) + 2 * S.n:] == 7.25).all()), (name, layout)
