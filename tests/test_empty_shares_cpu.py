"""What shares without blocks cost, in the CPU build (see test_cpu_build.py): their workgroups ask for query rows only in calls of one round."""
import pytest

from paper_2509_25224_amd import workloads as wl
from test_cpu_build import ADD, check, exe, run_cpu  # noqa: F401
from test_low_tiles_cpu import LOADS_OF_A_BLOCK, launch_info

LOADS_OF_HALF_A_WAVES_ROWS = 19 * 64


@pytest.mark.parametrize("shares,asking", [(128, 2 * 128), (140, 2)])   # of 40 rows each: 256 workgroups of 256 compute units, 280
def test_query_rows_of_shares_without_blocks(exe, tmp_path, shares, asking):
    case = wl.make_case("empty_shares", 107, batch=2, s_q=1, heads=40, seqlens=[64, 40], max_blocks_per_seq=150)
    out, lse, _ = run_cpu(exe, tmp_path, case, ADD, ns=shares)
    check(out, lse, case)
    tiles, _, loads = launch_info(tmp_path)
    assert tiles == 1   # (128 rows: not the library's own factor)
    assert loads == 2 * LOADS_OF_A_BLOCK + 2 * (asking + 2) * LOADS_OF_HALF_A_WAVES_ROWS   # two waves of four have rows
