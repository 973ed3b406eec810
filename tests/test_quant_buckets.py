"""Ordinary rows stay with the bucket sort: weights as fp32 draws, as a checkpoint's bf16 numbers (the smallest weight of
every group then scales to exactly 0), with half of them pruned to zero."""
import numpy as np
import pytest

from oracle import any4_quant_oracle
from paper_2507_04610_amd import inputs
from tests import quant_buckets


@pytest.mark.parametrize("bits,symmetric", ((4, False), (4, True), (2, False)))
@pytest.mark.parametrize("K", (1024, 4096, 5120, 8192, 14336))
@pytest.mark.parametrize("kind", ("fp32", "bf16", "pruned"))
def test_ordinary_rows_are_sorted_into_buckets(kind, K, bits, symmetric):
    qc = inputs.make_quant_case(16, K, bits, seed=K)
    w = qc.w
    if kind == "bf16":
        w = inputs.bf16_bits_to_f32(inputs.f32_to_bf16_bits(w))
    if kind == "pruned":
        if symmetric:
            pytest.skip("all zeros of a row in one bucket: the bitonic network's case")
        w = np.where(np.random.default_rng(K).random(w.shape) < 0.5, np.float32(0.0), w)
    for row in w:
        assert quant_buckets.accepted(any4_quant_oracle.scale_row(row, None, bits, symmetric)[2])
