"""The rule that sends a call's buckets to one workgroup (csrc/prefill.hip,
bucket_fits) against what that workgroup can hold, without a GPU: an expert may
take every token, and its running count over the 64-token chunks has 16 bits;
masks, counts, totals and offsets share at most 104 KB of LDS."""
import ctypes

import pytest

moeq = pytest.importorskip("paper_2509_25689_amd.moeq")


def _fits(n, k, E):
    f = moeq.lib._ZN4moeq11bucket_fitsEiii
    f.argtypes, f.restype = [ctypes.c_int] * 3, ctypes.c_bool
    return f(n, k, E)


@pytest.mark.parametrize("E", [1, 2, 4, 8, 10, 16, 64, 256, 1024])
def test_counts_and_lds_hold(E):
    sizes = {16, 64, 65, 2560, 2561, 65535, 65536, 65537, 70001, 1 << 17, 681472, 1 << 20}
    for k in (1, 2, 5, 6, 8, 32):
        if k > E:
            continue
        for n in sorted(sizes):
            if _fits(n, k, E):
                assert n <= 65535, (n, k, E)
                chunks = -(-n // 64)
                assert 10 * chunks * E + 4 * (2 * E + 1) <= 104 * 1024, (n, k, E)


def test_one_workgroup_serves_the_small_sizes():
    """Every call of 16 to 64 tokens, and the benchmark's 2048-token prefill."""
    for k, E in ((1, 1), (2, 16), (8, 256), (32, 1024)):
        assert all(_fits(n, k, E) for n in range(16, 65)), (k, E)
    assert _fits(2048, 8, 256) and _fits(65535, 2, 8)
