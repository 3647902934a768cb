"""Launch rules of the library at the edges where they change, asked from the library itself (host
code; no GPU)."""
import ctypes

import pytest


def _lib():
    from paper_1704_07559_amd import capi
    return capi._lib


@pytest.mark.parametrize("populations,rates,one_launch", [
    (0, 0, True), (1, 0, True), (4096, 4096, True),
    # HIP launches fewer than 2^32 threads along x: 2^24 - 1 blocks of 256 threads, 4096 bytes each
    (((1 << 24) - 1) * 4096, 0, True), (((1 << 24) - 1) * 4096 + 1, 0, False),
    (((1 << 24) - 2) * 4096, 4096, True), (((1 << 24) - 2) * 4096, 4097, False), (((1 << 24) - 2) * 4096 + 1, 2, False),
    # D3Q19 FP32 with its rate field: 858 and 859 million nodes, and the largest box there is
    (76 * 858_000_000, 4 * 858_000_000, True), (76 * 859_000_000, 4 * 859_000_000, False),
    (76 * ((1 << 30) - 1), 4 * ((1 << 30) - 1), False),
])
def test_state_copy_stays_within_one_launch(populations, rates, one_launch):
    f = _lib().lbm_internal_copy_is_one_launch
    f.argtypes, f.restype = [ctypes.c_size_t, ctypes.c_size_t], ctypes.c_int
    assert bool(f(populations, rates)) is one_launch
    blocks = -(-populations // 4096) - (-rates // 4096)
    assert (blocks * 256 < 1 << 32) is one_launch
