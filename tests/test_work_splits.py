"""Which split of the work the host code picks, where a wrong one costs time without making a result wrong.  The plans are pure
functions of the problem and of the number of compute units."""
import ctypes
import re

import pytest

from paper_2507_04610_amd import binding

CUS = 256


class StreamPlan(ctypes.Structure):          # csrc/any4_internal.h
    _fields_ = [("gw", ctypes.c_int), ("slabs", ctypes.c_int), ("slab_groups", ctypes.c_int), ("blocks_per_slab", ctypes.c_int),
                ("tiles", ctypes.c_int64), ("aux", ctypes.c_bool), ("workspace", ctypes.c_size_t)]


def plan_stream(M, N, K):
    f = binding.load_library()._ZN4any411plan_streamEllli          # any4::plan_stream(int64_t, int64_t, int64_t, int)
    f.restype, f.argtypes = StreamPlan, [ctypes.c_int64] * 3 + [ctypes.c_int]
    return f(M, N, K, CUS)


@pytest.mark.parametrize("M", (1, 8, 16))
@pytest.mark.parametrize("N", (40, 1000, 4096, 20685, 40000))
def test_no_wavefront_goes_through_groups_that_the_row_does_not_have(M, N):
    """up to 4096 weights a row the eight wavefronts have all of it between them, and a block goes through the row's groups rounded up to
    those of a wavefront of one, two or four, whichever is least (K = 640: five, not eight)"""
    for G in range(1, 33):
        p = plan_stream(M, N, 128 * G)
        least = min(-(-G // gw) * gw for gw in (1, 2, 4) if 8 * gw >= G)
        assert p.slabs == 1 and 8 * p.gw >= G
        assert p.slab_groups == least and p.slab_groups - G < p.gw, (G, p.gw, p.slab_groups)


@pytest.mark.parametrize("G", (5, 6, 7, 9, 10, 13, 14, 33, 34, 41, 42, 98, 101))
def test_who_loads_the_small_inputs(G):
    """shared: always for wavefronts of four groups, for others only while a block has few tiles; slabs then begin at whole fours"""
    for N in (16, 600, 2000, 4096, 4112, 9000, 16384, 16400, 31443):
        p = plan_stream(8, N, 128 * G)
        tpb = -(-p.tiles // p.blocks_per_slab)
        assert p.aux == (p.gw == 4 or tpb <= {1: 1, 2: 4}[p.gw]), (N, p.gw, tpb)
        if p.aux and p.slabs > 1:
            assert p.slab_groups % 4 == 0 and p.slab_groups <= 8 * p.gw
        assert (p.slabs - 1) * p.slab_groups < G <= p.slabs * p.slab_groups
    for rest in (1, 2, 3):
        assert not plan_stream(8, 600, 128 * rest).aux
    assert all(plan_stream(8, n, 128 * g).aux for n in (16, 40000) for g in (4, 8, 20, 32, 36, 100))


@pytest.mark.parametrize("N,K,slabs", ((92, 8832, 9), (34, 10112, 10), (66, 8448, 9), (36, 14080, 14), (32, 11520, 12), (19417, 12544, 4), (6668, 12544, 4)))
def test_few_tiles_are_spread_over_slabs_and_many_are_not(N, K, slabs):
    assert plan_stream(12, N, K).slabs == slabs


def test_rows_that_need_no_moving_have_kernels_without_it():
    """every variant that moves the last small inputs of a row down has one that does not, for K / 128 a multiple of 4"""
    names = {tuple(m) for m in re.findall(rb"decode_stream_kernelILi(\d)ELi(\d)ELb(\d)((?:ELb\d){5})ELb(\d)EEE", open(binding.LIB_PATH, "rb").read())}
    moving = {n for n in names if n[4] == b"1"}
    assert moving and all(n[2] == b"1" for n in moving)            # only where one wavefront loads for all
    assert {n[:4] + (b"0",) for n in moving} <= names


class PackPlan(ctypes.Structure):
    _fields_ = [("ok", ctypes.c_bool), ("mp", ctypes.c_int), ("passes", ctypes.c_int), ("tiles", ctypes.c_int64), ("nblocks", ctypes.c_int)]


def whole_k(M, N, K, bits):
    f = binding.load_library()._ZN4any49plan_packElllibi            # any4::plan_pack(int64_t, int64_t, int64_t, int, bool, int)
    f.restype, f.argtypes = PackPlan, [ctypes.c_int64] * 3 + [ctypes.c_int, ctypes.c_bool, ctypes.c_int]
    return f(M, N, K, bits, False, CUS).ok


@pytest.mark.parametrize("M,K,bits,tiles", ((1, 8320, 4, 64), (1, 16256, 3, 64), (1, 16512, 4, 128), (1, 28160, 4, 128), (2, 8064, 4, 16), (2, 13952, 3, 96),
                                            (3, 7680, 4, 64), (4, 4224, 3, 64), (1, 16512, 2, 48), (2, 13952, 2, 64)))
def test_few_tiles_are_not_given_a_whole_row_each(M, K, bits, tiles):
    """K no multiple of 1024: with that many tiles of 16 rows the blocks of the whole-K kernel leave most of the chip idle"""
    assert not whole_k(M, 16, K, bits) and not whole_k(M, 16 * tiles, K, bits)
    assert whole_k(M, 16 * tiles + 1, K, bits) and whole_k(M, 4096, K, bits)
    up = (K + 1023) // 1024 * 1024
    assert whole_k(M, 16, up, bits) == whole_k(M, 4096, up, bits)  # (whole kilos as they were: whatever the number of tiles)


@pytest.mark.parametrize("M,K,bits", ((1, 4224, 4), (1, 8064, 3), (1, 14464, 2), (2, 4224, 2), (4, 7680, 2)))
def test_short_rows_have_one_block_each_from_the_first_tile_on(M, K, bits):
    assert whole_k(M, 16, K, bits) and whole_k(M, 40000, K, bits)


def test_a_second_round_that_is_nearly_empty():
    """rows of more than 16384 weights and 257 .. 320 tiles: four compute units in five would wait for the others' second tile"""
    assert not whole_k(1, 4578, 24064, 4) and not whole_k(1, 5120, 16512, 3)
    assert whole_k(1, 4096, 24064, 4) and whole_k(1, 5121, 24064, 4) and whole_k(1, 4578, 12416, 4)


class BatchPlan(ctypes.Structure):
    _fields_ = [("ok", ctypes.c_bool), ("mt", ctypes.c_int), ("rows", ctypes.c_int), ("tiles_n", ctypes.c_int), ("slabs", ctypes.c_int),
                ("shared", ctypes.c_bool), ("counter_bytes", ctypes.c_size_t), ("sums_at", ctypes.c_size_t), ("workspace", ctypes.c_size_t),
                ("us", ctypes.c_double)]


class BatchPlans(ctypes.Structure):
    _fields_ = [("plain", BatchPlan), ("fine", BatchPlan)]


def plan_batch(M, N, K):
    f = binding.load_library()._ZN4any410plan_batchEllli            # any4::plan_batch(int64_t, int64_t, int64_t, int)
    f.restype, f.argtypes = BatchPlans, [ctypes.c_int64] * 3 + [ctypes.c_int]
    return f(M, N, K, CUS)


def test_adding_that_is_not_shared_is_not_priced_as_shared():
    """128 rows of x and K = 4096 in two slabs: 127 tiles of sums leave room for the words that slabs meet at, 128 do not, and one block adds all
    (0.3 - 0.4 us per MB of 33 instead of a meeting and 0.1)"""
    shared, alone = plan_batch(128, 127 * 256, 4096).plain, plan_batch(128, 128 * 256, 4096).plain
    assert (shared.slabs, shared.shared, shared.tiles_n) == (2, True, 127) and (alone.slabs, alone.shared, alone.tiles_n) == (2, False, 128)
    assert alone.us > shared.us + 2.0, (alone.us, shared.us)


@pytest.mark.parametrize("M,N,K", ((75, 9954, 640), (104, 12016, 640), (98, 9730, 512), (99, 9645, 512), (110, 7933, 512), (73, 8099, 512), (69, 12218, 896),
                                   (105, 4830, 384), (100, 24, 384), (39, 7466, 1024), (55, 6583, 1024), (45, 1425, 640)))
def test_short_rows_that_are_faster_in_one_piece_are_not_cut(M, N, K):
    """measured: in one piece 4 - 28 % faster than with the slabs that costs fitted to longer rows gave them"""
    assert plan_batch(M, N, K).plain.slabs == 1


@pytest.mark.parametrize("M,N,K", ((95, 42, 1024), (66, 30, 1024), (128, 4096, 1024), (64, 512, 1024), (64, 4096, 4096), (128, 6144, 4096)))
def test_rows_that_are_faster_cut_are_cut(M, N, K):
    assert plan_batch(M, N, K).plain.slabs > 1


class GemmPlan(ctypes.Structure):
    _fields_ = [("cus", ctypes.c_int), ("decode", ctypes.c_bool), ("stream", ctypes.c_bool), ("sp", StreamPlan), ("bp", BatchPlan),
                ("two_launches", ctypes.c_bool), ("bp_fine", BatchPlan), ("ksplit", ctypes.c_int), ("workspace", ctypes.c_size_t),
                ("counter_bytes", ctypes.c_size_t)]


def plan_gemm(M, N, K, bits=4):
    f = binding.load_library()._ZN4any49plan_gemmEllli              # any4::plan_gemm(int64_t, int64_t, int64_t, int)
    f.restype, f.argtypes = GemmPlan, [ctypes.c_int64] * 3 + [ctypes.c_int]
    return f(M, N, K, bits)


@pytest.mark.parametrize("bits", (4, 3, 2))
def test_two_launches_are_not_taken_where_one_is_faster(bits):
    """17 .. 24 rows of x: one launch of the kernel for a few dozen is faster (21 x 2736 x 2560 any3 re-laid-out 10.4 us, two launches 15.0) up to the
    sizes whose calls keep the bits of their two parts"""
    for M in range(17, 25):
        for N, K in ((1312, 2560), (2736, 2560), (3013, 2560), (1500, 3072), (2048, 4096), (3824, 4096), (4096, 3584), (4097, 4096), (4096, 4224)):
            p = plan_gemm(M, N, K, bits)
            assert p.bp.ok and not p.two_launches, (M, N, K)
        assert plan_gemm(M, 4000, 4096, bits).two_launches and plan_gemm(M, 4096, 4096, bits).two_launches
    assert not plan_gemm(25, 4000, 4096, bits).two_launches and not plan_gemm(16, 4000, 4096, bits).two_launches
