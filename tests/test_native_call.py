"""The native GEMM call (csrc/any4_torch.cpp) against the checked Python call it stands in for: the same bits on
every format, and a plain "no" - never an answer - to whatever the Python call refuses."""
import pytest
import torch

import paper_2507_04610_amd as any4
from paper_2507_04610_amd import binding, inputs


def problem(M, N, K, bits, f16=False, device="cuda"):
    t = inputs.make_case_device(M, N, K, bits, seed=5, device=device, f16=f16)
    return t, torch.randint(-2 ** 31, 2 ** 31 - 1, (N, K * bits // 32), dtype=torch.int32, device=device)


def test_host_tensors_are_left_to_the_checked_call():
    t, codes = problem(1, 32, 256, 4, device="cpu")
    any4.load_library()
    assert binding._native_gemm(t["x"], codes, t["lut"], t["scale"], t["offset"], 4, None, None, 128, False) is None
    with pytest.raises(any4.Any4Error, match="device memory"):
        any4.any4_gemm(t["x"], codes, t["lut"], t["scale"], t["offset"], 4)


@pytest.mark.gpu
@pytest.mark.parametrize("M,bits,kind", [(1, 4, "table"), (3, 3, "table"), (1, 2, "one"), (20, 4, "int4"), (1, 4, "group64"),
                                         (17, 4, "f16"), (300, 4, "table"), (2, 4, "repacked")])
def test_native_call_gives_the_bits_of_the_checked_call(M, bits, kind):
    N, K = 83, 8192 if kind == "repacked" else 5120
    t, codes = problem(M, N, K, bits, f16=kind == "f16")
    lut = {"one": t["lut"][:1].contiguous(), "int4": None}.get(kind, t["lut"])
    scale, offset, group = t["scale"], t["offset"], 128
    if kind == "group64":
        group = 64
        scale, offset = (v.repeat_interleave(2, dim=1).contiguous() for v in (scale, offset))
    if kind == "repacked":
        codes = any4.any4_repack(codes, bits)
    entry = "any4_gemm_repacked" if kind == "repacked" else "any4_gemm" if group == 128 else "any4_gemm_grouped"
    want = binding._gemm(entry, t["x"], codes, N, lut, scale, offset, bits, None, None, None if group == 128 else group)
    got = binding._native_gemm(t["x"], codes, lut, scale, offset, bits, None, None, group, kind == "repacked")
    assert got.dtype == want.dtype and torch.equal(got.view(torch.int16), want.view(torch.int16))
    out = torch.empty_like(want)
    ws = torch.empty(max(16, any4.any4_gemm_workspace_bytes(M, N, K, bits)), dtype=torch.uint8, device="cuda")
    assert binding._native_gemm(t["x"], codes, lut, scale, offset, bits, out, ws, group, kind == "repacked") is out
    assert torch.equal(out.view(torch.int16), want.view(torch.int16))


@pytest.mark.gpu
def test_refusals_name_the_mistake():
    t, codes = problem(2, 64, 512, 4)
    x, lut, s, o = t["x"], t["lut"], t["scale"], t["offset"]
    for args, words in (((x[:, ::2], codes, lut, s, o), "contiguous"), ((x.float(), codes, lut, s, o), "dtype"),
                        ((x, codes, lut, s[:, :1].contiguous(), o), "scale must have shape"),
                        ((x, codes, lut[:3].contiguous(), s, o), "lut must have shape")):
        with pytest.raises(any4.Any4Error, match=words):
            any4.any4_gemm(*args, 4)
    with pytest.raises(any4.Any4Error, match="workspace"):
        any4.any4_gemm(torch.cat([x] * 200), codes, lut, s, o, 4, workspace=torch.empty(16, dtype=torch.uint8, device="cuda"))
