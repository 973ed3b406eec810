"""The matrix-core kernel (more than 128 rows of x) at the edges of its tiles (256 rows of x, 128 rows of weights, 64 values
along K): one group, group counts that leave its rings of three part-filled, offsets in and out of 16-byte pieces, rows of y
that are and are not whole 16-byte pieces, K slices, rows so long that addresses take 64 bits, and the
longest before that.  Against the oracle; bar as in test_gpu_parity.py."""
import numpy as np
import pytest

from paper_2507_04610_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = [(129, 1, 1), (256, 128, 2), (257, 264, 3), (130, 127, 33), (385, 520, 40), (512, 136, 72), (777, 129, 23)]
LONG = [(129, 24, 1026)]          # K = 131328


def dev16(a, f16=False):
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
    for M, N, G in SHAPES + LONG:
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


# The longest rows of the kernels with 32-bit offsets, and just beyond (64-bit addresses).  Two blocks of rows of x and of weights.
LONGEST = 1 << 25
LONG_M, LONG_N = 257, 136


@pytest.fixture(scope="module")
def long_x():
    t = torch.zeros(LONG_M * (LONGEST + 128), dtype=torch.int16, device="cuda")
    yield t
    del t
    torch.cuda.empty_cache()


@pytest.mark.parametrize("K", (LONGEST, LONGEST + 128))
@pytest.mark.parametrize("variant,bits", (("plain", 4), ("plain", 3), ("plain", 2), ("repack", 4), ("repack", 3), ("f16", 4), ("g64", 4), ("g64", 2), ("int4", 4)))
def test_longest_rows(oracle, long_x, variant, bits, K):
    """All activations are 0 but those of some groups (the first, the last, both sides of the K slices' ends, others),
    so that the oracle needs these groups only; the others add exactly 0."""
    import paper_2507_04610_amd as any4
    any4.load_library()
    M, N, G, f16, per = LONG_M, LONG_N, K // 128, variant == "f16", 2 if variant == "g64" else 1
    rng = np.random.default_rng(bits)
    ends = np.array([s * G // 8 for s in range(1, 8)])
    at = np.unique(np.concatenate(([0, 1, G - 2, G - 1], ends - 1, ends, rng.integers(0, G, 20))))
    cs = inputs.make_case(M, N, 128 * len(at), bits, seed=bits, f16=f16)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(bits)
    codes = torch.empty((N, K * bits // 32), dtype=torch.int32, device="cuda").random_(-2 ** 31, 2 ** 31 - 1, generator=gen)
    dt = torch.float16 if f16 else torch.bfloat16
    scale = torch.empty((N, per * G), device="cuda").uniform_(0.005, 0.02, generator=gen).to(dt)
    offset = torch.empty((N, per * G), device="cuda").normal_(0, 0.002, generator=gen).to(dt)
    lut = cs.lut
    if variant == "int4":
        lut = np.tile(inputs.f32_to_bf16_bits(np.arange(-8, 8, dtype=np.float32)), (N, 1))
    groups = torch.from_numpy(at).cuda()
    x = long_x[:M * K].view(M, G, 128)
    x[:, groups] = torch.from_numpy(cs.x.view(np.int16)).cuda().view(M, -1, 128)
    words = lambda t: np.ascontiguousarray(t.view(N, G, -1)[:, groups].cpu().view(torch.int16 if t.dtype == dt else torch.int32).numpy()).reshape(N, -1)
    y64 = oracle.gemm(cs.x, words(codes).view(np.uint32), lut, words(scale).view(np.uint16), words(offset).view(np.uint16), 128 * len(at), bits,
                      threads=8, group=128 // per, f16=f16)
    print((variant, bits, M, N, K), flush=True)
    xs = x.view(M, K).view(dt)
    if variant == "repack":
        y = any4.any4_gemm_repacked(xs, any4.any4_repack(codes, bits), dev16(lut), scale, offset, bits)
    else:
        y = any4.any4_gemm(xs, codes, None if variant == "int4" else dev16(lut, f16), scale, offset, bits, group=128 // per)
    x[:, groups] = 0
    got = y.float().cpu().numpy().astype(np.float64)
    tol = 1e-2 * oracle.rms(y64) + np.abs(y64) * (2.0 ** -11 if f16 else 2.0 ** -8)
    assert np.all(np.abs(got - y64) <= tol), float((np.abs(got - y64) - tol).max())


@pytest.mark.parametrize("N", (136, 131))
def test_outputs_round_to_nearest_even(oracle, N):
    """One activation per row of x, no offsets: an output is the product of three bf16 numbers, exact in fp32 while it is a
    normal number, so that only its rounding to bf16 is left.  With results from sub-normal to beyond bf16's range."""
    import paper_2507_04610_amd as any4
    any4.load_library()
    M, K, bits = 300, 256, 4
    rng = np.random.default_rng(N)
    cs = inputs.make_case(M, N, K, bits, seed=N)
    at = rng.integers(0, K, M)
    value = inputs.f32_to_bf16_bits((rng.standard_normal(M) * 2.0 ** rng.integers(-70, 66, M)).astype(np.float32))
    x = np.zeros((M, K), np.uint16)
    x[np.arange(M), at] = value
    scale = inputs.f32_to_bf16_bits((rng.uniform(1, 2, cs.scale.shape) * 2.0 ** rng.integers(-72, 72, cs.scale.shape)).astype(np.float32))
    y = any4.any4_gemm(dev16(x), any4.any4_pack(torch.from_numpy(cs.codes_u8).cuda(), bits), dev16(cs.lut), dev16(scale),
                       dev16(np.zeros_like(cs.offset)), bits)
    f64 = lambda a: inputs.bf16_bits_to_f32(a).astype(np.float64)
    w = np.take_along_axis(f64(cs.lut), cs.codes_u8.astype(np.int64), axis=1) * np.repeat(f64(scale), 128, axis=1)
    exact = f64(value)[:, None] * w[:, at].T
    with np.errstate(over="ignore"):
        want = torch.from_numpy(exact.astype(np.float32)).to(torch.bfloat16).float().numpy()
    assert np.isinf(want).any() and (np.abs(want[want != 0]) < 2.0 ** -126).any()
    assert np.array_equal(y.float().cpu().numpy(), want)


@pytest.mark.parametrize("group", (128, 64))
@pytest.mark.parametrize("slices", (2, 3, 4, 5, 6, 7, 8))
def test_slices_meet_in_parts(oracle, slices, group):
    """A few tiles, cut along K into every number of slices there is; the words that count arrivals hold zeros and
    garbage at first.  Every result has the same bits."""
    import paper_2507_04610_amd as any4
    any4.load_library()
    M, N, G, bits = 300, 264, 4 * slices + (slices < 8), 4                   # (at least four groups a slice)
    K = 128 * G
    cs = inputs.make_case(M, N, K, bits, seed=slices)
    sc, of = cs.scale, cs.offset
    if group == 64:
        sc, of = (np.ascontiguousarray(np.repeat(a, 2, axis=1)) for a in (sc, of))
    packed = oracle.pack(cs.codes_u8, bits)
    y64 = oracle.gemm(cs.x, packed, cs.lut, sc, of, K, bits, threads=8, group=group)
    args = (dev16(cs.x), torch.from_numpy(packed.view(np.int32)).cuda(), dev16(cs.lut), dev16(sc), dev16(of), bits)
    need = any4.any4_gemm_workspace_bytes(M, N, K, bits)
    tiles = 2 * 3
    assert need == (M * ((4 * G + 15) // 16 * 16) * 2 + 255) // 256 * 256 + 256 + tiles * slices * 256 * 128 * 4
    first = None
    for word in (0, 0xA5A5A5A5A5A5A5, -1):
        ws = torch.full((need // 8,), word, dtype=torch.int64, device="cuda").view(torch.uint8)
        for _ in range(4):
            y = any4.any4_gemm(*args, group=group, workspace=ws)
            if first is None:
                first = y.clone()
                got = y.float().cpu().numpy().astype(np.float64)
                assert np.all(np.abs(got - y64) <= 1e-2 * oracle.rms(y64) + np.abs(y64) * 2.0 ** -8)
            assert torch.equal(y.view(torch.int16), first.view(torch.int16))


@pytest.mark.parametrize("K", (384, 1152))                                   # whole tiles, two slices
@pytest.mark.parametrize("variant,bits,N", (("plain", 4, 136), ("plain", 3, 131), ("g64", 4, 131), ("f16", 4, 136), ("int4", 4, 131), ("repack", 2, 136)))
def test_not_finite(variant, bits, N, K):
    """A NaN or an infinity in a row of x makes that row of y NaN (the group sum's low part is none), one among the scales or
    offsets of a row of weights leaves that column of y without a finite number; every other output has the bits that it
    has without them.  In first, inner and last groups, in the last rows (which stand in for those past the end)."""
    import paper_2507_04610_amd as any4
    any4.load_library()
    M, f16, group = 300, variant == "f16", 64 if variant == "g64" else 128
    cs = inputs.make_case(M, N, K, bits, seed=K + N, f16=f16)
    sc, of = (np.ascontiguousarray(np.repeat(a, 128 // group, axis=1)) for a in (cs.scale, cs.offset))
    codes = any4.any4_pack(torch.from_numpy(cs.codes_u8).cuda(), bits)
    lut = None if variant == "int4" else dev16(cs.lut, f16)

    def gemm(x, s, o):
        if variant == "repack":
            return any4.any4_gemm_repacked(dev16(x), any4.any4_repack(codes, bits), lut, dev16(s), dev16(o), bits)
        return any4.any4_gemm(dev16(x, f16), codes, lut, dev16(s, f16), dev16(o, f16), bits, group=group)
    clean = gemm(cs.x, sc, of)
    inf = 0x7C00 if f16 else 0x7F80
    nan, ninf = inf | 0x40, inf | 0x8000
    x = cs.x.copy()
    rows = {3: (0, nan), 64: (K - 1, inf), 200: (K // 2 + 5, ninf), 255: (130, nan), M - 1: (K - 130, inf)}
    for m, (k, v) in rows.items():
        x[m, k] = v
    s, o = sc.copy(), of.copy()
    s[5, 0], s[70, -1], s[N - 1, 1] = nan, inf, nan
    o[9, -1], o[40, 0], o[129, 2] = nan, inf, ninf
    y = gemm(x, s, o)
    bad = torch.zeros((M, N), dtype=torch.bool, device="cuda")
    bad[:, [5, 9, 40, 70, 129, N - 1]] = True
    bad[list(rows)] = True
    assert torch.equal(~torch.isfinite(y), bad)
    assert torch.isnan(y[list(rows)]).all() and torch.isnan(y[:, [5, 9, N - 1]]).all()
    assert torch.equal(y[~bad].view(torch.int16), clean[~bad].view(torch.int16))
