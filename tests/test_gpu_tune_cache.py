"""The SpMV choice of one mesh is not taken for another on the other side of the line from which the product
from the cells is offered (3 million stored entries).  The line lies inside a bucket of sizes: 64^2 and
76^2 cells of degree 2 share one.
"""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CHILD = """
import sys, torch
torch.cuda.set_device(0)
import paper_2105_11993_amd as thm
from tests._gpu_helpers import spec
for m in map(int, sys.argv[1:]):
    S = thm.thm_assemble(spec(2, m, 2, 9.0))
    thm.thm_apply_operator(S, torch.ones(S.n, dtype=torch.complex128, device="cuda"))
    print("variant", m, S.info["nnz"], S.fresh_info()["spmv_variant"], flush=True)
"""


def variants(tmp_path, cached, *cells):
    f = tmp_path / "tune"
    f.write_text("".join(f"gfx950:d2:p2:n16:b1:g1:{p} {cached}\n" for p in ("fp64", "fp32")))
    r = subprocess.run([sys.executable, "-c", CHILD, *map(str, cells)], cwd=ROOT, capture_output=True, text=True,
                       timeout=100, env=dict(os.environ, THM_TUNE_CACHE=str(f)))
    print(r.stdout, r.stderr, flush=True)
    assert r.returncode == 0
    out = [line.split() for line in r.stdout.splitlines() if line.startswith("variant")]
    return {int(w[1]): (int(w[2]), int(w[3])) for w in out}


def test_line_inside_a_bucket(tmp_path):
    # an assembled form of 32 lanes a row, as a mesh below the line may have left it
    v = variants(tmp_path, 321, 64, 76)
    assert v[64][0] < 3000000 <= v[76][0]
    assert v[64][1] == 321 and v[76][1] != 321
    # the cells, as a mesh above the line may have left them in the same bucket
    v = variants(tmp_path, 30, 64)
    assert v[64][1] != 30
