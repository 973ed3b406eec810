"""The kernel for one to four rows of x that walks the whole K axis inside one block, K no multiple of 1024, from the number of tiles
on at which it is taken: every number of register sets, whose last unit and piece of scales are there in part, all code widths
and both code layouts; and the calls just below that number, which the streaming kernel takes.  Bar as in test_gpu_parity.py."""
import pytest
from test_gpu_small_m_whole_k import any4, run          # noqa: F401  (any4 is a fixture)

from paper_2507_04610_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", (4, 3, 2))
@pytest.mark.parametrize("M,N,G", [(1, 1025, 65), (1, 1024, 65), (1, 1040, 94), (1, 1025, 97), (1, 1057, 126), (1, 2049, 131), (1, 2048, 131), (1, 2049, 163),
                                   (1, 2060, 187), (1, 2049, 221), (1, 2053, 255), (2, 257, 33), (2, 256, 61), (2, 1537, 70), (2, 1536, 94), (2, 1540, 127),
                                   (3, 1025, 33), (4, 1024, 35), (4, 1030, 63), (3, 1090, 46)])
def test_both_sides_of_the_line(any4, oracle, bits, M, N, G):          # noqa: F811
    run(any4, oracle, M, N, 128 * G, bits, seed=inputs.case_seed(74, bits, G % 10))
