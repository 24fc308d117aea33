"""What shares without blocks cost, in the CPU build (see test_cpu_build.py): their workgroups ask for query rows only in calls of one round, and calls
of more shares or workers than blocks, which are cut like the library's own, are not launched as that many on lower row tiles."""
import pytest

from paper_2509_25224_amd import workloads as wl
from test_cpu_build import ADD, BALANCED, MUL, check, exe, launch_info, run_cpu  # noqa: F401
from test_low_tiles_cpu import LOADS_OF_A_BLOCK

LOADS_OF_HALF_A_WAVES_ROWS = 19 * 64


@pytest.mark.parametrize("shares,asking", [(128, 2 * 128), (140, 2)])   # of 40 rows each: 256 workgroups of 256 compute units, 280
def test_query_rows_of_shares_without_blocks(exe, tmp_path, shares, asking):
    case = wl.make_case("empty_shares", 107, batch=2, s_q=1, heads=40, seqlens=[64, 40], max_blocks_per_seq=150)
    out, lse, _ = run_cpu(exe, tmp_path, case, ADD, ns=shares)
    check(out, lse, case)
    tiles, _, loads, _ = launch_info(tmp_path)
    assert tiles == 1   # (128 rows: not the library's own factor)
    assert loads == 2 * LOADS_OF_A_BLOCK + 2 * (asking + 2) * LOADS_OF_HALF_A_WAVES_ROWS   # two waves of four have rows


@pytest.mark.parametrize("heads,lens,flags,ns,tiles,workgroups", [
    (128, [64, 1], 0, 35, 1, 2 * 35), (128, [64, 1], 0, 27, 4, 2 * 27 * 4), (128, [64], BALANCED, 70, 1, 70),   # a block at most: the library's own is no cut
    (24, [50 * 64 - 7, 640], 0, 100, 2, 2 * 50 * 2), (100, [320, 30], BALANCED, 200, 7, 10 * 7),   # a block each: launched as that
    (24, [450, 576], 0, 100, 1, 2 * 100)])                                                   # the library would not cut these
def test_more_shares_than_blocks(exe, tmp_path, heads, lens, flags, ns, tiles, workgroups):
    case = wl.make_case("many_shares", 108, batch=len(lens), s_q=1, heads=heads, seqlens=lens)
    out, lse, splits = run_cpu(exe, tmp_path, case, MUL, flags=flags, ns=ns)
    assert splits == ns
    check(out, lse, case)
    got_tiles, _, _, got_workgroups = launch_info(tmp_path)
    assert (got_tiles, got_workgroups) == (tiles, -(-workgroups // 8) * 8)
