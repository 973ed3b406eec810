"""The scratch of 17 <= M <= 128 rows of x stays within the library's own (any4_gemm_noalloc refuses what exceeds it)."""
import pytest

from paper_2507_04610_amd import binding


@pytest.mark.parametrize("M", (17, 33, 64, 65, 97, 128))
@pytest.mark.parametrize("bits", (4, 3, 2))
def test_workspace_fits_the_librarys_scratch(M, bits):
    lib = binding.load_library()
    for N in (1, 4097, 28672, 57344, 128256, 300000):
        for K in (128, 4096, 8192, 14336, 28672, 65536):
            assert lib.any4_gemm_workspace_bytes(M, N, K, bits) <= binding.NOALLOC_SCRATCH_BYTES, (M, N, K)
