"""Up to 16 rows of x, rows of 5 .. 14 and of 33 and more groups, no multiple of 4: wavefronts of one and of two groups, whose
small inputs one of them loads for all (few tiles a block) or each reads itself (many), on both sides of each line, every storage
variant, against the oracle.  Bar as in test_gpu_parity.py."""
import numpy as np
import pytest

from paper_2507_04610_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# M, N, groups: one tile a block / two; four tiles a block / five; slabs of both kinds
PROBLEMS = ((16, 4096, 5), (2, 4097, 5), (5, 333, 7), (1, 4113, 7), (3, 16384, 6), (9, 16385, 6), (1, 700, 9), (16, 2000, 10), (4, 8200, 13),
            (7, 50, 14), (2, 16500, 14), (5, 600, 33), (16, 9000, 33), (8, 5400, 41), (3, 1377, 98))


def dev16(a, f16):
    t = torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).cuda()
    return t.view(torch.float16 if f16 else torch.bfloat16)


@pytest.mark.parametrize("bits", (4, 3, 2))
@pytest.mark.parametrize("variant", ("plain", "repack", "f16", "g64", "g256", "one_table", "int4"))
def test_few_groups(oracle, bits, variant):
    import paper_2507_04610_amd as any4
    any4.load_library()
    if variant == "int4" and bits != 4:
        pytest.skip("the table-free format has 4 bits")
    f16, group = variant == "f16", {"g64": 64, "g256": 256}.get(variant, 128)
    for M, N, G in PROBLEMS:
        if group == 256 and G % 2:
            continue
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
        y64 = oracle.gemm(cs.x, packed, lut, sc, of, K, bits, threads=16, group=group, f16=f16)
        codes = torch.from_numpy(packed.view(np.int32)).cuda()
        x, s, o = dev16(cs.x, f16), dev16(sc, f16), dev16(of, f16)
        print((bits, variant, M, N, K), flush=True)
        if variant == "repack":
            y = any4.any4_gemm_repacked(x, any4.any4_repack(codes, bits), dev16(lut, f16), s, o, bits)
        else:
            t = None if variant == "int4" else dev16(lut[:1] if variant == "one_table" else lut, f16)
            y = any4.any4_gemm(x, codes, t, s, o, bits, group=group)
        tol = 1e-2 * oracle.rms(y64) + np.abs(y64) * (2.0 ** -11 if f16 else 2.0 ** -8)
        assert np.all(np.abs(y.float().cpu().numpy().astype(np.float64) - y64) <= tol), (M, N, K)
