"""The default entry (no split factor given) on batches whose lengths make it take ranges instead of equal shares, and on
batches where it stays with equal shares: the library's source compiled for the host (see test_cpu_build.py), under
AddressSanitizer with a workspace of exactly the documented size, against the oracle."""
import numpy as np
import pytest

from paper_2509_25224_amd import workloads as wl
from test_cpu_build import check, exe, run_cpu  # noqa: F401


def prefers_ranges(case, splits, capacity):
    nb = -(-case.seqlens.astype(np.int64) // 64)
    shares = case.batch * splits
    workers = min(capacity, shares * 2052 // 1028 - case.batch + 1)
    return nb.sum() / workers + 12 < -(-shares // capacity) * (nb.max() / splits + 6)


LONG_AND_EMPTY = [0] * 20 + [5000] + [40, 0] * 9 + [64, 65, 129] + [0] * 18   # one long sequence between short and empty ones


@pytest.mark.parametrize("heads,s_q,lens,ranges,variant,flags,static",
                         [(16, 1, LONG_AND_EMPTY, True, 1, 0, False), (3, 1, LONG_AND_EMPTY, True, 0, 32, True),
                          (129, 1, [5000] + [0, 63] * 15, True, 2, 0, False), (16, 1, [600, 0, 520], False, 1, 0, False)])
def test_default_decomposition(exe, tmp_path, heads, s_q, lens, ranges, variant, flags, static):
    case = wl.make_case("ranges", 83, batch=len(lens), s_q=s_q, heads=heads, seqlens=lens, spare_frac=0.1)
    out, lse, splits = run_cpu(exe, tmp_path, case, variant, flags=flags, static_ws=static)
    assert splits > 1
    assert prefers_ranges(case, splits, 256 // -(-heads * s_q // 128)) == ranges
    check(out, lse, case)
