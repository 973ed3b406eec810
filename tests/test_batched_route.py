"""Which kernel serves 17 .. 128 rows of x: the one for a few dozen rows, two launches of the streaming kernel (up to
24 rows, matrices with one tile of weights per block) or the matrix-core kernel, by their expected times."""
import numpy as np
import pytest

from paper_2507_04610_amd import binding, inputs


def test_few_tiles_do_not_pay_for_slabs():
    # 4 blocks with 8 steps (23.7 us) or, cut in two along K, 8 blocks with 4 steps and a meeting of their sums (28.6 us)
    assert binding.load_library().any4_gemm_workspace_bytes(128, 1024, 1024, 4) == 0


@pytest.mark.gpu
@pytest.mark.parametrize("variant", ("any4", "any3", "any2", "repack", "f16", "g256", "one_table", "int4", "g64"))
@pytest.mark.parametrize("M", (17, 24, 25))
def test_two_streaming_launches(oracle, variant, M):
    """4000 x 4096: up to 24 rows the bits of the streaming kernel on the first 16 rows and on the rest - but not
    without a table and not with groups of 64 - and on either route the oracle's values"""
    import torch
    import paper_2507_04610_amd as any4
    N, K = 4000, 4096
    bits = {"any3": 3, "any2": 2}.get(variant, 4)
    f16, group = variant == "f16", {"g64": 64, "g256": 256}.get(variant, 128)
    cs = inputs.make_case(M, N, K, bits, seed=M + bits, f16=f16)
    lut, sc, of = cs.lut, cs.scale, cs.offset
    if variant == "int4":
        lut = np.tile(inputs.f32_to_bf16_bits(np.arange(-8, 8, dtype=np.float32)), (N, 1))
    if variant == "one_table":
        lut = np.ascontiguousarray(np.tile(cs.lut[:1], (N, 1)))
    if group == 64:
        sc, of = (np.ascontiguousarray(np.repeat(a, 2, axis=1)) for a in (sc, of))
    elif group == 256:
        sc, of = np.ascontiguousarray(sc[:, ::2]), np.ascontiguousarray(of[:, ::2])

    def dev(a):
        t = torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).cuda()
        return t.view(torch.float16 if f16 else torch.bfloat16)
    packed = oracle.pack(cs.codes_u8, bits)
    codes = torch.from_numpy(packed.view(np.int32)).cuda()
    x, t = dev(cs.x), None if variant == "int4" else dev(lut[:1] if variant == "one_table" else lut)
    s, o = dev(sc), dev(of)

    def gemm(rows):
        if variant == "repack":
            return any4.any4_gemm_repacked(rows, any4.any4_repack(codes, bits), t, s, o, bits)
        return any4.any4_gemm(rows, codes, t, s, o, bits, group=group)
    y = gemm(x)
    y64 = oracle.gemm(cs.x, packed, lut, sc, of, K, bits, threads=8, group=group, f16=f16)
    tol = 1e-2 * oracle.rms(y64) + np.abs(y64) * (2.0 ** -11 if f16 else 2.0 ** -8)
    assert np.all(np.abs(y.float().cpu().numpy().astype(np.float64) - y64) <= tol)
    apart = torch.cat((gemm(x[:16].contiguous()), gemm(x[16:].contiguous())))
    if variant != "f16":                                          # (fp16: whichever is expected to be faster)
        assert torch.equal(y.view(torch.int16), apart.view(torch.int16)) == (M <= 24 and variant not in ("int4", "g64"))


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K,repacked", ((20, 4000, 4096, False), (40, 1000, 14336, True), (80, 99000, 8192, False)))
def test_captured_calls(M, N, K, repacked):
    """two streaming launches, K slabs, several launches in one workspace: every replay of a captured call gives the eager
    call's bits, with eager work in between and the output overwritten"""
    import torch
    import paper_2507_04610_amd as any4
    t = inputs.make_case_device(M, N, K, 4, seed=M)
    codes = any4.any4_pack(t["codes_u8"], 4)
    del t["codes_u8"]
    if repacked:
        codes = any4.any4_repack(codes, 4)
    gemm = any4.any4_gemm_repacked if repacked else any4.any4_gemm
    y = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
    ws = torch.full((max(16, any4.any4_gemm_workspace_bytes(M, N, K, 4)),), 0xA5, dtype=torch.uint8, device="cuda")
    run = lambda: gemm(t["x"], codes, t["lut"], t["scale"], t["offset"], 4, out=y, workspace=ws)
    want = run().clone()
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        run()
    for _ in range(4):
        y.fill_(9.0)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y.view(torch.int16), want.view(torch.int16))
        assert torch.equal(run().view(torch.int16), want.view(torch.int16))
