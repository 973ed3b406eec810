"""Matrices whose sums of K slabs do not fit the library's scratch at 17 .. 128 rows of x: the kernel for a few dozen
rows takes them in several launches that share the workspace."""
import numpy as np
import pytest

from paper_2507_04610_amd import binding, inputs


@pytest.mark.parametrize("M,N,K", ((128, 57344, 8192), (97, 57344, 8192), (128, 6144, 28672), (112, 128256, 4096), (80, 100000, 8192),
                                   (48, 100000, 8192), (64, 49000, 14336)))
def test_large_sums_do_not_leave_the_kernel(M, N, K):
    """the workspace is one counter and `slabs` tiles of fp32 sums per tile of a launch, not the matrix-core kernel's"""
    need = binding.load_library().any4_gemm_workspace_bytes(M, N, K, 4)
    rows, bn = (M + 31) // 32 * 32, 128 if M <= 64 else 256
    assert need <= binding.NOALLOC_SCRATCH_BYTES
    sizes = {(8 * t + 255) // 256 * 256 + t * s * rows * bn * 4 for s in range(2, 65) for t in range(1, (N + bn - 1) // bn + 1)}
    assert need in sizes


@pytest.mark.gpu
@pytest.mark.parametrize("M,G,variant", ((128, 47, "plain"), (97, 32, "repack"), (65, 61, "g64"), (80, 64, "f16"), (100, 30, "one_table"),
                                         (128, 24, "int4"), (64, 64, "any3"), (112, 40, "any2"), (48, 64, "repack")))
def test_several_launches(oracle, M, G, variant):
    """300 rows of weights over and over, so that the oracle has only those to do, and a number of rows that leaves the
    last launch and its last tile ragged; twice in a row in the same memory"""
    import torch
    import paper_2507_04610_amd as any4
    bits = {"any3": 3, "any2": 2}.get(variant, 4)
    f16, group = variant == "f16", 64 if variant == "g64" else 128
    rows, times, K = 300, 330, 128 * G
    N = rows * times
    cs = inputs.make_case(M, rows, K, bits, seed=M, f16=f16)
    lut, sc, of = cs.lut, cs.scale, cs.offset
    if variant == "int4":
        lut = np.tile(inputs.f32_to_bf16_bits(np.arange(-8, 8, dtype=np.float32)), (rows, 1))
    if variant == "one_table":
        lut = np.ascontiguousarray(np.tile(cs.lut[:1], (rows, 1)))
    if group == 64:
        other = inputs.make_case(1, rows, K, bits, seed=M + 7)
        sc = np.ascontiguousarray(np.stack([sc, other.scale], axis=2).reshape(rows, -1))
        of = np.ascontiguousarray(np.stack([of, other.offset], axis=2).reshape(rows, -1))
    packed = oracle.pack(cs.codes_u8, bits)
    y64 = oracle.gemm(cs.x, packed, lut, sc, of, K, bits, threads=8, group=group, f16=f16)

    def dev(a):
        t = torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).cuda()
        return t.view(torch.float16 if f16 else torch.bfloat16)
    many = lambda t: t.repeat(times, 1)
    codes = many(torch.from_numpy(packed.view(np.int32)).cuda())
    t = None if variant == "int4" else dev(lut[:1]) if variant == "one_table" else many(dev(lut))
    x, s, o = dev(cs.x), many(dev(sc)), many(dev(of))
    need = any4.any4_gemm_workspace_bytes(M, N, K, bits)
    tile = (M + 31) // 32 * 32 * (128 if M <= 64 else 256) * 4
    assert 0 < need < 2 * tile * (N // (128 if M <= 64 else 256)), "one launch would do"
    ws = torch.full((need,), 0xA5, dtype=torch.uint8, device="cuda")
    if variant == "repack":
        codes = any4.any4_repack(codes, bits)
        run = lambda: any4.any4_gemm_repacked(x, codes, t, s, o, bits, workspace=ws)
    else:
        run = lambda: any4.any4_gemm(x, codes, t, s, o, bits, group=group, workspace=ws)
    y = run()
    want = torch.from_numpy(y64).cuda()[:, None, :]
    tol = 1e-2 * oracle.rms(y64) + want.abs() * (2.0 ** -11 if f16 else 2.0 ** -8)
    assert bool(((y.view(M, times, rows).double() - want).abs() <= tol).all())
    assert torch.equal(y.view(torch.int16), run().view(torch.int16))
