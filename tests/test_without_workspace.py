"""17 .. 128 rows of x and short rows of weights: calls that have always gone without a workspace still do when the caller brings none
or a smaller one than is asked for, in one piece along K; what needed one is refused without it."""
import numpy as np
import pytest

from paper_2507_04610_amd import binding, inputs

# M, N, K: first and later tiles from which such calls have needed none, at every tile height
GO = ((32, 1, 640), (17, 4000, 768), (20, 1300, 1024), (32, 3900, 1280), (25, 9000, 1536), (64, 100, 640), (33, 3600, 1024), (50, 2000, 1280), (96, 700, 512),
      (65, 2000, 896), (80, 600, 1024), (96, 3100, 1152), (128, 1100, 512), (97, 4000, 1024), (128, 300, 1152), (100, 2000, 1280),
      (33, 16400, 3200))
STAY = ((32, 1280, 1024), (32, 3800, 1280), (64, 1800, 1152), (64, 4096, 4096), (96, 500, 1024), (96, 3000, 1152), (128, 15000, 1152), (128, 1700, 1280),
        (128, 4096, 1536), (128, 40000, 1536), (60, 4096, 3200), (32, 40000, 16384), (129, 512, 512), (200, 4096, 4096), (16, 64, 8192))


def goes_without(M, N, K):
    import ctypes
    f = binding.load_library()._ZN4any418batch_goes_withoutElll     # any4::batch_goes_without(int64_t, int64_t, int64_t)
    f.restype, f.argtypes = ctypes.c_bool, [ctypes.c_int64] * 3
    return f(M, N, K)


def test_which():
    lib = binding.load_library()
    assert all(goes_without(*p) for p in GO) and not any(goes_without(*p) for p in STAY)
    assert all(lib.any4_gemm_workspace_bytes(*p, 4) > 0 for p in STAY)
    assert sum(lib.any4_gemm_workspace_bytes(*p, 4) > 0 for p in GO) >= 10        # (the others need none in any case)


def test_refused_before_anything_is_touched():
    lib, A = binding.load_library(), 0x1000
    for M, N, K in STAY:
        need = lib.any4_gemm_workspace_bytes(M, N, K, 4)
        assert lib.any4_gemm(A, A, A, A, A, M, N, K, 4, A, None, 0, None) == -5
        assert lib.any4_gemm(A, A, A, A, A, M, N, K, 4, A, A, need - 1, None) == -5
        assert lib.any4_gemm_grouped(A, A, A, A, A, M, N, K, 4, 64, A, None, 0, None) == -5


@pytest.mark.gpu
@pytest.mark.parametrize("variant", ("plain", "repack", "f16", "g64", "g256", "one_table", "int4"))
def test_served(oracle, variant):
    import torch
    lib = binding.load_library()
    import paper_2507_04610_amd as any4
    f16, group = variant == "f16", {"g64": 64, "g256": 256}.get(variant, 128)
    for M, N, K in GO:
        if K % group:
            continue
        cs = inputs.make_case(M, N, K, 4, seed=M + N % 91, f16=f16)
        lut, sc, of = cs.lut, cs.scale, cs.offset
        if variant == "int4":
            lut = np.tile(inputs.f32_to_bf16_bits(np.arange(-8, 8, dtype=np.float32)), (N, 1))
        if variant == "one_table":
            lut = np.ascontiguousarray(np.tile(cs.lut[:1], (N, 1)))
        if group == 64:
            other = inputs.make_case(1, N, K, 4, seed=M + 7)
            sc = np.ascontiguousarray(np.stack([sc, other.scale], axis=2).reshape(N, -1))
            of = np.ascontiguousarray(np.stack([of, other.offset], axis=2).reshape(N, -1))
        elif group == 256:
            sc, of = np.ascontiguousarray(sc[:, ::2]), np.ascontiguousarray(of[:, ::2])
        packed = oracle.pack(cs.codes_u8, 4)
        y64 = oracle.gemm(cs.x, packed, lut, sc, of, K, 4, threads=16, group=group, f16=f16)
        tol = 1e-2 * oracle.rms(y64) + np.abs(y64) * (2.0 ** -11 if f16 else 2.0 ** -8)

        def dev(a):
            t = torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).cuda()
            return t.view(torch.float16 if f16 else torch.bfloat16)
        codes = torch.from_numpy(packed.view(np.int32)).cuda()
        if variant == "repack":
            codes = any4.any4_repack(codes, 4)
        x, t, s, o = dev(cs.x), dev(lut[:1] if variant == "one_table" else lut), dev(sc), dev(of)
        y = torch.full((M, N), 9.0, dtype=x.dtype, device="cuda")
        small = torch.full((256,), 0xA5, dtype=torch.uint8, device="cuda")
        args = [x.data_ptr(), codes.data_ptr(), None if variant == "int4" else t.data_ptr(), s.data_ptr(), o.data_ptr(), M, N, K, 4]
        entry = {"repack": "any4_gemm_repacked", "f16": "any4_gemm_f16", "one_table": "any4_gemm_single_table"}.get(variant, "any4_gemm")
        if group != 128:
            entry, args = "any4_gemm_grouped", args + [group]
        print((variant, M, N, K), flush=True)
        for ws, n in ((None, 0), (small.data_ptr(), 16)):
            y.fill_(9.0)
            assert getattr(lib, entry)(*args, y.data_ptr(), ws, n, torch.cuda.current_stream().cuda_stream) == 0
            torch.cuda.synchronize()
            assert np.all(np.abs(y.float().cpu().numpy().astype(np.float64) - y64) <= tol), (M, N, K)
        assert bool((small == 0xA5).all())
