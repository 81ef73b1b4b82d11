"""Rules by which the host sizes and shapes launches, called in the library
without a GPU (they touch no device)."""
import ctypes
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    return ctypes.CDLL(os.path.join(ROOT, "paper_2306_07212_amd", "libpcx.so"))


def test_weight_gradient_chunks_stay_short(lib):
    """A chunk is summed in FP32 by the FP32 backward: fewer than 4096 vertices, or a 256th of them, whatever the
    layer's tiles."""
    chunks = lib["_ZN3pcx10bwd_chunksEiii"]  # pcx::bwd_chunks(int, int, int)
    for N, K in ((1, 3), (64, 64), (200, 65), (256, 256)):
        for Vs in (1, 63, 64, 4095, 4096, 100_000, 131_073, 524_287, 524_288, 1_400_000, 5_000_000, 2**31 - 1):
            n = chunks(Vs, N, K)
            assert n >= 1 and -(-Vs // n) <= max(4095, -(-Vs // 256)), (N, K, Vs, n)
            assert n <= 1024 and (n == 1 or Vs // n >= 64)
