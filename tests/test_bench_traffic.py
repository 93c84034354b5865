"""The measured HBM traffic of the tree products is reported only while the sources that hold them are those
of the record (no GPU)."""
import hashlib
import json
import os
import shutil

import pytest

from tests.test_bench_contract import ROOT, _bench_module

CSRC = os.path.join("paper_2105_11993_amd", "csrc")


@pytest.fixture
def bench(tmp_path):
    mod = _bench_module()
    (tmp_path / "profiles").mkdir()
    (tmp_path / CSRC).mkdir(parents=True)
    for name in os.listdir(os.path.join(ROOT, CSRC)):
        shutil.copy(os.path.join(ROOT, CSRC, name), tmp_path / CSRC / name)
    mod.ROOT = str(tmp_path)
    return mod


def digest(bench, name):
    return hashlib.sha256(open(os.path.join(bench.ROOT, CSRC, name), "rb").read()).hexdigest()


@pytest.mark.parametrize("name", ["k_bcr_mfma_c2_traffic.json", "k_nd_mfma_c2_traffic.json"])
@pytest.mark.parametrize("kernel", ["k_nd_mfma<float>", "k_bcr_mfma<float,4>"])
def test_record_tied_to_another_source_is_not_used(bench, kernel, name):
    """kernels_prec.hip holds the layered forms' kernel, not the tree products."""
    rec = {"kernel": kernel, "hbm_bytes_per_launch": 7.0e7, "kernels_prec_sha256": digest(bench, "kernels_prec.hip")}
    open(os.path.join(bench.ROOT, "profiles", name), "w").write(json.dumps(rec))
    assert bench.measured_traffic(63.5e6) is None


@pytest.mark.parametrize("changed", ["kernels_nd.hip", "nd.cpp", "nd.h"])
def test_record_of_the_tree_products(bench, changed):
    rec = {"kernel": "k_nd_mfma<float>", "hbm_bytes_per_launch": 1.0e7,
           "sources": {n: digest(bench, n) for n in ("kernels_nd.hip", "nd.cpp", "nd.h")}}
    open(os.path.join(bench.ROOT, "profiles", "k_nd_mfma_c2_traffic.json"), "w").write(json.dumps(rec))
    assert bench.measured_traffic(63.5e6) == 1.0e7
    with open(os.path.join(bench.ROOT, CSRC, changed), "a") as f:
        f.write("\n")
    assert bench.measured_traffic(63.5e6) is None
