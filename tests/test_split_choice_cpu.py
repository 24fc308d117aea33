"""The library's own split factor (num_splits 0) and shares without blocks, in the host code and the CPU build (see test_cpu_build.py)."""
import numpy as np
import pytest

from paper_2509_25224_amd import amla, workloads as wl
from test_cpu_build import ADD, COMP, MUL, TRANSPOSED, check, exe, run_cpu  # noqa: F401


@pytest.mark.parametrize("rows", [1, 16, 17, 32, 33, 128, 129, 256, 512])
def test_chosen_factor_is_bounded(rows):
    """Never more shares than blocks; where one round of workgroups holds them all (256 compute units without a device) the partial
    rows fit the static array, so that no call that it used to hold is refused; the transposed family has the coarse factor."""
    s_q, heads = (rows // 128, 128) if rows % 128 == 0 else (1, rows)
    tiles = -(-rows // 128)
    for batch in (1, 2, 3, 7, 16, 33, 64, 100, 255, 300):
        for blocks in (1, 2, 4, 7, 8, 16, 17, 24, 64, 100, 256, 1000, 4096):
            d = amla.make_desc(batch, s_q, heads, 20000, blocks)
            ns = amla.amla_effective_splits(d)
            assert 1 <= ns <= min(blocks, 256) and (ns == 1 or batch * tiles < 256)
            if batch * tiles * ns <= 256:
                assert amla.amla_workspace_bytes(d) <= amla.amla_static_workspace_limit()
            coarse = amla.amla_effective_splits(amla.make_desc(batch, s_q, heads, 20000, blocks, flags=amla.AMLA_FLAG_TRANSPOSED_ACC))
            assert coarse <= max(1, blocks // 4) and (batch * tiles * coarse <= 256 or coarse == ns)
            if rows > 32 and blocks <= 16:
                assert ns <= max(1, blocks // 4)


@pytest.mark.parametrize("heads,variant,flags,ns", [(40, ADD, 0, 9), (8, MUL, 0, 70), (130, COMP, 0, 5), (40, ADD, TRANSPOSED, 9)])
def test_shares_without_blocks(exe, tmp_path, heads, variant, flags, ns):
    """More shares than a sequence has blocks, among them 70 (a workgroup merges a row then) and sequences with none: the workspace
    comes filled with NaN, so a partial row that nobody wrote must not count."""
    case = wl.make_case("shares", 89, batch=4, s_q=1, heads=heads, seqlens=[200, 0, 64, 330], spare_frac=0.2)
    out, lse, _ = run_cpu(exe, tmp_path, case, variant, flags=flags, ns=ns)
    check(out, lse, case)
    assert np.all(out[1] == 0) and np.all(np.isneginf(lse[1]))


# (nb blocks in W shares: share w holds none while floor((w + 1) nb / W) = floor(w nb / W), so the first ones are the empty ones)
@pytest.mark.parametrize("heads,lens,variant,flags,ns", [
    (32, [64], ADD, TRANSPOSED, 256), (32, [100], MUL, TRANSPOSED, 256), (128, [64, 300], ADD, TRANSPOSED, 65),
    (128, [64, 0] + [64] * 6 + [30 * 64], ADD, 0, 65),
    (64, [128], COMP, TRANSPOSED, 129), (1100, [128, 300], MUL, 0, 129), (43, [192], ADD, TRANSPOSED, 193), (3200, [192], ADD, 0, 193),
    (8, [128, 64, 0], ADD, TRANSPOSED, 129)])
def test_first_64_shares_without_blocks(exe, tmp_path, heads, lens, variant, flags, ns):
    """A wave merges 64 shares at a time: sequences whose first 64 hold nothing, one block each, two and three, in calls that do
    not take the workgroup-per-row merge; all but the last have so many partial rows that the lengths are looked at first."""
    case = wl.make_case("late_shares", 94, batch=len(lens), s_q=1, heads=heads, seqlens=lens, spare_frac=0.2)
    n_rows = len(lens) * heads
    assert flags == TRANSPOSED or n_rows > 16 * ns
    assert (n_rows * ns >= 8192) == (heads != 8)
    out, lse, _ = run_cpu(exe, tmp_path, case, variant, flags=flags, ns=ns)
    check(out, lse, case)
