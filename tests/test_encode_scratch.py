"""The encoder's scratch (CPU only): at most 42 bytes per Gaussian beyond the digit counts
of its sort, which take a byte per Gaussian at most and a fixed part below a
megabyte, so that sets which fit beside two copies of their codes and a sort's four
arrays still do."""
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2603_20611_amd", "libgaussianpile.so")


@pytest.mark.skipif(not os.path.exists(LIB), reason="library not built")
@pytest.mark.parametrize("n", [1, 2049, 500_000, 100_000_000, (1 << 31) - 1])
def test_bytes_per_gaussian(n):
    from paper_2603_20611_amd import binding as B
    need = B.load().gp_encode_scratch(n)
    assert 0 < need <= 43 * n + (1 << 20)
