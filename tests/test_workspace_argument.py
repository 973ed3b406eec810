"""A caller's workspace is written by the kernels: what is not one piece of x's device memory is refused by name,
in the native call and in the checked one."""
import pytest
import torch

import paper_2507_04610_amd as any4
from paper_2507_04610_amd import binding, inputs

M, N, K = 4, 64, 16384          # K slabs: needs a workspace


def bad(t):
    return {"host": t.cpu(), "expanded": t[:1].expand(t.numel()), "strided": torch.cat((t, t)).view(t.numel(), 2)[:, 0]}


@pytest.mark.parametrize("kind", ("expanded", "strided"))
def test_gaps_and_repeats_are_refused(kind):
    with pytest.raises(any4.Any4Error, match="one piece"):
        binding._scratch(bad(torch.zeros(4096, dtype=torch.uint8))[kind], torch.device("cpu"))


def test_another_device_is_refused():
    with pytest.raises(any4.Any4Error, match="x's device"):
        binding._scratch(torch.zeros(4096, dtype=torch.uint8), torch.device("cuda", 0))
    with pytest.raises(any4.Any4Error, match="x's device"):
        binding._scratch(bytearray(4096), torch.device("cuda", 0))


@pytest.mark.parametrize("shape,dtype", (((4096,), torch.uint8), ((16, 64), torch.float32), ((0,), torch.uint8)))
def test_one_piece_is_taken_whatever_its_type(shape, dtype):
    t = torch.zeros(shape, dtype=dtype)
    for v in (t, t.t()) if t.dim() == 2 else (t,):
        assert binding._scratch(v, torch.device("cpu")) == (v.data_ptr(), t.numel() * t.element_size())


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ("host", "expanded", "strided"))
def test_gemm_refuses_it(kind):
    t = inputs.make_case_device(M, N, K, 4, seed=3)
    codes = any4.any4_pack(t["codes_u8"], 4)
    good = torch.empty(any4.any4_gemm_workspace_bytes(M, N, K, 4), dtype=torch.uint8, device="cuda")
    args = (t["x"], codes, t["lut"], t["scale"], t["offset"], 4)
    assert binding._native_gemm(*args, None, bad(good)[kind], 128, False) is None
    with pytest.raises(any4.Any4Error, match="workspace must be"):
        any4.any4_gemm(*args, workspace=bad(good)[kind])
    assert torch.equal(any4.any4_gemm(*args, workspace=good).view(torch.int16), any4.any4_gemm(*args).view(torch.int16))
