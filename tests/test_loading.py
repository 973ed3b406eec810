"""libany4.so alone is enough: without the torch extension (not built, or built for another torch) every entry point
is there and GEMM calls take the checked path, with one warning."""
import os
import subprocess
import sys

import pytest
import torch

import paper_2507_04610_amd as any4
from paper_2507_04610_amd import binding, inputs

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

WITHOUT = """
import sys, warnings
sys.modules["paper_2507_04610_amd._any4_torch"] = None        # what makes its import raise ImportError
import torch
import paper_2507_04610_amd as any4
from paper_2507_04610_amd import binding, inputs
with warnings.catch_warnings(record=True) as caught:
    warnings.simplefilter("always")
    assert any4.any4_version() >= 100 and any4.any4_gemm_workspace_bytes(4, 64, 16384, 4) > 0
    any4.load_library()
assert [w.category for w in caught] == [RuntimeWarning], caught
"""
HOST = """
t = inputs.make_case_device(1, 32, 256, 4, seed=5, device="cpu")
codes = torch.zeros((32, 32), dtype=torch.int32)
try:
    any4.any4_gemm(t["x"], codes, t["lut"], t["scale"], t["offset"], 4)
    raise SystemExit("host tensors were taken")
except any4.Any4Error as e:
    assert "device memory" in str(e)
"""
def run(code):
    r = subprocess.run([sys.executable, "-c", WITHOUT + code], cwd=ROOT, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr


def test_without_the_extension():
    run(HOST)


@pytest.mark.gpu
@pytest.mark.parametrize("M,repacked", ((1, False), (20, False), (2, True)))
def test_gemm_without_the_extension(M, repacked, monkeypatch):
    any4.load_library()
    t = inputs.make_case_device(M, 83, 5120, 4, seed=5)
    codes = any4.any4_pack(t["codes_u8"], 4)
    args = (t["x"], any4.any4_repack(codes, 4) if repacked else codes, t["lut"], t["scale"], t["offset"], 4)
    gemm = any4.any4_gemm_repacked if repacked else any4.any4_gemm
    want = gemm(*args)
    monkeypatch.setattr(binding, "_native_gemm", binding._no_native_gemm)
    assert torch.equal(gemm(*args).view(torch.int16), want.view(torch.int16))
