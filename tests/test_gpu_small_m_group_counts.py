"""Up to 16 rows of x with numbers of groups that are no multiple of 4, whose last scales of a row are loaded together
with earlier ones and moved down: one to eleven groups, K slabs that end with one to three, one and several tiles of rows
per block, every storage variant, against the oracle.  Bar as in test_gpu_parity.py."""
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
def test_numbers_of_groups(oracle, bits, variant):
    import paper_2507_04610_amd as any4
    any4.load_library()
    if variant == "int4" and bits != 4:
        pytest.skip("the table-free format has 4 bits")
    f16, group = variant == "f16", {"g64": 64, "g256": 256}.get(variant, 128)
    # (33 .. 35 groups of 33 rows: five slabs, the last of one to three groups; 20500 rows: six tiles a block)
    for M, N, G in ((1, 17, 1), (2, 33, 2), (4, 16, 3), (1, 33, 5), (16, 100, 6), (3, 31, 7), (7, 4200, 9), (2, 20500, 5), (9, 48, 11),
                    (1, 33, 33), (16, 33, 34), (5, 33, 35), (4, 40, 66), (6, 5003, 22), (2, 50, 37), (1, 17, 70)):
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
        x, o = dev16(cs.x, f16), dev16(of, f16)
        print((bits, variant, M, N, K), flush=True)

        def run(s):
            if variant == "repack":
                return any4.any4_gemm_repacked(x, any4.any4_repack(codes, bits), dev16(lut, f16), s, o, bits)
            t = None if variant == "int4" else dev16(lut[:1] if variant == "one_table" and N > 1 else lut, f16)
            return any4.any4_gemm(x, codes, t, s, o, bits, group=group)
        s = dev16(sc, f16)
        y = run(s)
        got = y.float().cpu().numpy().astype(np.float64)
        tol = 1e-2 * oracle.rms(y64) + np.abs(y64) * (2.0 ** -11 if f16 else 2.0 ** -8)
        assert np.all(np.abs(got - y64) <= tol), (M, N, K, float((np.abs(got - y64) - tol).max()))
        s[N // 2] = float("nan")                                  # a row's scales are its own: the others keep their bits
        z = run(s)
        keep = torch.arange(N, device="cuda") != N // 2
        assert torch.equal(z[:, keep].view(torch.int16), y[:, keep].view(torch.int16)), (M, N, K)
        assert bool(z[:, N // 2].isnan().all())
