"""Where the K slabs of 17 .. 128 rows of x, and the K slices of more, meet: the blocks of a tile share the adding, wait for each other for a while
and otherwise leave their part to the last.  Two to more than eight slabs, parts of unequal size, every tile height, whatever
the workspace held, with another stream's work on the GPU that keeps some blocks from running at the same time: the bits of
the first call every time, and the oracle's values."""
import numpy as np
import pytest

from paper_2507_04610_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TAG = 0x24B47C5EED17 << 17          # csrc/any4_splitk.h
CASES = ((17, 200, 2048), (32, 1100, 4096), (48, 4096, 4096), (64, 6144, 4096), (64, 5003, 8192), (40, 300, 14336), (90, 700, 2944),
         (96, 4096, 14336), (65, 2000, 5120), (128, 3000, 4096), (128, 6144, 4096), (113, 257, 8192),
         (129, 512, 4096), (200, 4096, 4096), (300, 1000, 2944), (512, 6144, 4096), (777, 2900, 2944), (1030, 700, 2048))


def dev_bf16(a_u16):
    return torch.from_numpy(np.ascontiguousarray(a_u16).view(np.int16)).cuda().view(torch.bfloat16)


@pytest.mark.parametrize("M,N,K", CASES)
def test_meetings(oracle, M, N, K):
    import paper_2507_04610_amd as any4
    any4.load_library()
    cs = inputs.make_case(M, N, K, 4, seed=M + N % 89)
    packed = oracle.pack(cs.codes_u8, 4)
    need = any4.any4_gemm_workspace_bytes(M, N, K, 4)
    rows, bn = ((M + 31) // 32 * 32, 128 if M <= 64 else 256) if M <= 128 else (256, 128)
    assert need > rows * bn * 4 * 2, "these problems are cut along K"
    x, codes = dev_bf16(cs.x), torch.from_numpy(packed.view(np.int32)).cuda()
    lut, sc, of = dev_bf16(cs.lut), dev_bf16(cs.scale), dev_bf16(cs.offset)
    y = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
    rng = np.random.default_rng(M + N)
    marked = torch.full((need // 8,), TAG | 0xFF00, dtype=torch.int64, device="cuda").view(torch.uint8)      # every part said to be left
    turned = torch.full((need // 8,), TAG | 1 << 16, dtype=torch.int64, device="cuda").view(torch.uint8)
    many = torch.full((need // 8,), TAG | 0xFF, dtype=torch.int64, device="cuda").view(torch.uint8)          # more arrivals than slabs
    fills = (torch.zeros(need, dtype=torch.uint8, device="cuda"), torch.full((need,), 0xA5, dtype=torch.uint8, device="cuda"),
             torch.from_numpy(rng.integers(0, 256, need, dtype=np.uint8)).cuda(), marked, turned, many)
    side = torch.cuda.Stream()
    a = torch.randn(1024, 1024, device="cuda")
    first = None
    for busy in (False, True):
        for i, fill in enumerate(fills):
            ws = fill.clone()
            ws = torch.cat([ws, ws.new_zeros(need - ws.numel())]) if ws.numel() < need else ws
            torch.cuda.synchronize()
            if busy:
                with torch.cuda.stream(side):
                    for _ in range(10):
                        a @ a
            for rep in range(12):
                y.fill_(9.0)
                any4.any4_gemm(x, codes, lut, sc, of, 4, out=y, workspace=ws)
                got = y.view(torch.int16).cpu()
                if first is None:
                    first = got.clone()
                    y64 = oracle.gemm(cs.x, packed, cs.lut, cs.scale, cs.offset, K, 4, threads=16)
                    tol = 1e-2 * oracle.rms(y64) + np.abs(y64) * 2.0 ** -8
                    assert np.all(np.abs(y.float().cpu().numpy().astype(np.float64) - y64) <= tol), (M, N, K)
                assert torch.equal(first, got), (M, N, K, busy, i, rep)
            torch.cuda.synchronize()
