"""What the choice of kernel by M leaves to chance elsewhere: the matrix-core kernel (M > 128) at one and two groups in
every storage variant; guard bands around, and arbitrary workspace contents under, the kernel for 17 .. 128 rows; one
decoder layer at full size there; the native call on a stream of its own and with an unaligned tensor."""
import numpy as np
import pytest
import torch

import test_gpu_guard_words as guard_words
import test_gpu_splitk_workspace as splitk_workspace
from paper_2507_04610_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def any4():
    import paper_2507_04610_amd as lib
    lib.load_library()
    return lib


def dev16(a, f16):
    t = torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).cuda()
    return t.view(torch.float16 if f16 else torch.bfloat16)


@pytest.mark.parametrize("bits", (4, 3, 2))
@pytest.mark.parametrize("variant", ("plain", "repack", "f16", "g64", "g256", "one_table", "int4"))
def test_matrix_core_kernel_at_few_groups(any4, oracle, bits, variant):
    if variant == "int4" and bits != 4:
        pytest.skip("the table-free format has 4 bits")
    f16, group = variant == "f16", {"g64": 64, "g256": 256}.get(variant, 128)
    for M, N, K in ((129, 128, 128), (129, 1, 256), (200, 200, 256), (256, 129, 128), (257, 127, 384)):
        if K % group:
            continue
        cs = inputs.make_case(M, N, K, bits, seed=inputs.case_seed(31, bits, M % 10), f16=f16)
        lut, sc, of = cs.lut, cs.scale, cs.offset
        if variant == "int4":
            lut = np.tile(inputs.f32_to_bf16_bits(np.arange(-8, 8, dtype=np.float32)), (N, 1))
        if variant == "one_table":
            lut = np.ascontiguousarray(np.tile(cs.lut[:1], (N, 1)))
        if group == 64:
            other = inputs.make_case(1, N, K, bits, seed=M + N)
            sc = np.ascontiguousarray(np.stack([sc, other.scale], axis=2).reshape(N, -1))
            of = np.ascontiguousarray(np.stack([of, other.offset], axis=2).reshape(N, -1))
        elif group == 256:
            sc, of = np.ascontiguousarray(sc[:, ::2]), np.ascontiguousarray(of[:, ::2])
        packed = oracle.pack(cs.codes_u8, bits)
        y64 = oracle.gemm(cs.x, packed, lut, sc, of, K, bits, threads=8, group=group, f16=f16)
        codes = torch.from_numpy(packed.view(np.int32)).cuda()
        x, s, o = dev16(cs.x, f16), dev16(sc, f16), dev16(of, f16)
        t = None if variant == "int4" else dev16(lut[:1] if variant == "one_table" and N > 1 else lut, f16)
        y = any4.any4_gemm_repacked(x, any4.any4_repack(codes, bits), t, s, o, bits) if variant == "repack" else \
            any4.any4_gemm(x, codes, t, s, o, bits, group=group)
        got = y.float().cpu().numpy().astype(np.float64)
        tol = 1e-2 * oracle.rms(y64) + np.abs(y64) * (2.0 ** -11 if f16 else 2.0 ** -8)
        assert np.all(np.abs(got - y64) <= tol), (M, N, K)


@pytest.mark.parametrize("M,N,K,bits,variant", [
    (200, 200, 256, 4, "f16"), (140, 200, 1024, 4, "no_table"), (129, 130, 4096, 2, "repacked"),            # matrix cores
    (24, 4000, 4096, 4, "plain"), (17, 4001, 4096, 3, "repacked"),                                          # two streaming launches
    (31, 100, 14336, 4, "repacked"), (64, 333, 4224, 4, "group64"), (96, 257, 8192, 3, "f16"), (128, 257, 4096, 2, "plain"),
    (100, 100, 2048, 4, "group256"), (65, 200, 1024, 4, "no_table"), (33, 1, 128, 3, "plain"), (97, 127, 640, 4, "group64")])
def test_gemm_writes_only_y_and_its_workspace(any4, oracle, M, N, K, bits, variant):
    guard_words.test_gemm_writes_only_y_and_its_workspace(any4, oracle, M, N, K, bits, variant)


@pytest.mark.parametrize("M,N,K,bits", [(20, 100, 14336, 4), (40, 300, 8192, 3), (96, 257, 8192, 2), (128, 520, 14336, 4)])
def test_slabs_at_17_to_128_rows_whatever_the_workspace_held(any4, oracle, M, N, K, bits):
    splitk_workspace.test_result_does_not_depend_on_what_the_workspace_held(any4, oracle, M, N, K, bits)


@pytest.mark.parametrize("N,K", list(inputs.LLAMA3_8B_SHAPES.values()))
@pytest.mark.parametrize("M", (24, 64, 128))
def test_decoder_layer_at_full_size(any4, M, N, K):
    """every output against the fp64 product with the dequantised weights (which are bit for bit the oracle's)"""
    t = inputs.make_case_device(M, N, K, 4, seed=N % 97 + M)
    codes = any4.any4_pack(t["codes_u8"], 4)
    y = any4.any4_gemm(t["x"], codes, t["lut"], t["scale"], t["offset"], 4)
    want = t["x"].double() @ any4.any4_dequant(codes, t["lut"], t["scale"], t["offset"], K, 4).double().t()
    # half a bf16 unit of output rounding and the fp32 sums of K products
    err = (y.double() - want).abs() - want.abs() * 2.0 ** -8
    assert float(err.max()) <= 1e-3 * float(want.pow(2).mean().sqrt())


@pytest.mark.parametrize("M", (1, 16, 40, 200))
def test_native_call_runs_on_the_current_stream(any4, M):
    t = inputs.make_case_device(M, 300, 8192, 4, seed=M)
    codes = any4.any4_pack(t["codes_u8"], 4)
    want = any4.any4_gemm(t["x"], codes, t["lut"], t["scale"], t["offset"], 4)
    x = torch.zeros_like(t["x"])
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        torch.cuda._sleep(2000000)                      # about a millisecond: on another stream the call would see zeros
        x.copy_(t["x"])
        y = any4.any4_gemm(x, codes, t["lut"], t["scale"], t["offset"], 4)
    side.synchronize()
    assert torch.equal(y.view(torch.int16), want.view(torch.int16))


@pytest.mark.parametrize("name", ("x", "lut", "scale", "offset", "out", "workspace"))
def test_native_call_refuses_unaligned_tensors(any4, name):
    t = inputs.make_case_device(4, 64, 16384, 4, seed=2)
    t["codes"] = any4.any4_pack(t["codes_u8"], 4)
    t["out"] = torch.full((4, 64), 7.0, dtype=torch.bfloat16, device="cuda")
    t["workspace"] = torch.empty(any4.any4_gemm_workspace_bytes(4, 64, 16384, 4), dtype=torch.uint8, device="cuda")
    src = t[name]
    raw = torch.zeros(src.numel() + 16, dtype=src.dtype, device="cuda")
    t[name] = raw[1:1 + src.numel()].view(src.shape).copy_(src)
    with pytest.raises(any4.Any4Error, match="16-byte aligned"):
        any4.any4_gemm(t["x"], t["codes"], t["lut"], t["scale"], t["offset"], 4, out=t["out"], workspace=t["workspace"])
    torch.cuda.synchronize()
    assert bool((t["out"] == 7.0).all()) or name == "out"
