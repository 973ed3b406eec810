"""The kernel for 17 .. 128 rows of x at the edges of its tiles (32 rows of x, 128 / 256 rows of weights), with one
group, group counts that leave k parts without work, K slabs of unequal length and every storage variant,
against the oracle.  Bar as in test_gpu_parity.py."""
import numpy as np
import pytest

from paper_2507_04610_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def dev16(a, f16):
    t = torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).cuda()
    return t.view(torch.float16 if f16 else torch.bfloat16)


@pytest.mark.parametrize("bits", (4, 3, 2))
@pytest.mark.parametrize("variant", ("plain", "repack", "f16", "g64", "g256", "one_table", "int4"))
def test_tile_edges(oracle, bits, variant):
    import paper_2507_04610_amd as any4
    any4.load_library()
    if variant == "int4" and bits != 4:
        pytest.skip("the table-free format has 4 bits")
    f16, group = variant == "f16", {"g64": 64, "g256": 256}.get(variant, 128)
    for M, N, G in ((17, 1, 1), (32, 129, 3), (33, 127, 32), (64, 300, 22), (65, 255, 7), (96, 257, 40), (97, 31, 9), (128, 520, 33)):
        if group == 256 and G % 2:
            G += 1
        K = 128 * G
        cs = inputs.make_case(M, N, K, bits, seed=M + G, f16=f16)
        lut, sc, of = cs.lut, cs.scale, cs.offset
        if variant == "int4":
            lut = np.tile(inputs.f32_to_bf16_bits(np.arange(-8, 8, dtype=np.float32)), (N, 1))
        if variant == "one_table":
            lut = np.ascontiguousarray(np.tile(cs.lut[:1], (N, 1)))
        if group == 64:
            other = inputs.make_case(1, N, K, bits, seed=M + G + 7)
            sc = np.ascontiguousarray(np.stack([sc, other.scale], axis=2).reshape(N, -1))
            of = np.ascontiguousarray(np.stack([of, other.offset], axis=2).reshape(N, -1))
        elif group == 256:
            sc, of = np.ascontiguousarray(sc[:, ::2]), np.ascontiguousarray(of[:, ::2])
        packed = oracle.pack(cs.codes_u8, bits)
        y64 = oracle.gemm(cs.x, packed, lut, sc, of, K, bits, threads=8, group=group, f16=f16)
        codes = torch.from_numpy(packed.view(np.int32)).cuda()
        x, s, o = dev16(cs.x, f16), dev16(sc, f16), dev16(of, f16)
        print((bits, variant, M, N, K), flush=True)
        ws = torch.full((max(16, any4.any4_gemm_workspace_bytes(M, N, K, bits)),), 0xA5, dtype=torch.uint8, device="cuda")

        def run():
            if variant == "repack":
                return any4.any4_gemm_repacked(x, any4.any4_repack(codes, bits), dev16(lut, f16), s, o, bits, workspace=ws)
            t = None if variant == "int4" else dev16(lut[:1] if variant == "one_table" and N > 1 else lut, f16)
            return any4.any4_gemm(x, codes, t, s, o, bits, group=group, workspace=ws)
        y = run()
        got = y.float().cpu().numpy().astype(np.float64)
        tol = 1e-2 * oracle.rms(y64) + np.abs(y64) * (2.0 ** -11 if f16 else 2.0 ** -8)
        assert np.all(np.abs(got - y64) <= tol), (M, N, K, float((np.abs(got - y64) - tol).max()))
        assert torch.equal(y.view(torch.int16), run().view(torch.int16))     # the workspace is left clean


@pytest.mark.parametrize("M,group", ((33, 128), (64, 128), (50, 64)))
def test_many_rows_of_weights_without_slabs(oracle, M, group):
    """so many rows of weights that sums of K slabs would not fit the library's scratch: blocks of 32 rows of x, no
    slabs, no workspace.  300 rows of weights over and over, so that the oracle has only those to do."""
    import paper_2507_04610_amd as any4
    lib = any4.load_library()
    rows, times, K, bits = 300, 330, 128 * 47, 4
    N = rows * times
    assert lib.any4_gemm_workspace_bytes(M, N, K, bits) == 0
    cs = inputs.make_case(M, rows, K, bits, seed=M)
    sc, of = cs.scale, cs.offset
    if group == 64:
        sc, of = (np.ascontiguousarray(np.repeat(a, 2, axis=1)) for a in (sc, of))
    packed = oracle.pack(cs.codes_u8, bits)
    y64 = oracle.gemm(cs.x, packed, cs.lut, sc, of, K, bits, threads=8, group=group)
    many = lambda t: t.repeat(times, 1)
    y = any4.any4_gemm(dev16(cs.x, False), many(torch.from_numpy(packed.view(np.int32)).cuda()), many(dev16(cs.lut, False)),
                       many(dev16(sc, False)), many(dev16(of, False)), bits, group=group)
    # (every copy against the oracle, not against each other: a block's first step along K, and so the order of its
    # sums, depends on its place among the blocks)
    want = torch.from_numpy(y64).cuda()[:, None, :]
    tol = 1e-2 * oracle.rms(y64) + want.abs() * 2.0 ** -8
    assert bool(((y.view(M, times, rows).double() - want).abs() <= tol).all())
