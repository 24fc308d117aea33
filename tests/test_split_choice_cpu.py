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


@pytest.mark.parametrize("rows", [1, 16, 32, 33, 40, 128, 256, 512])
def test_short_tables_are_not_cut(rows):
    """What the coarse factor (the transposed family's) leaves whole stays whole: no workspace, and results of any BF16 magnitude,
    where partial rows are FP16."""
    s_q, heads = (rows // 128, 128) if rows % 128 == 0 else (1, rows)
    for batch in (1, 2, 5, 6, 14, 64, 128, 129, 255, 300):
        for blocks in range(1, 70):
            d = amla.make_desc(batch, s_q, heads, 20000, blocks)
            if amla.amla_effective_splits(amla.make_desc(batch, s_q, heads, 20000, blocks, flags=amla.AMLA_FLAG_TRANSPOSED_ACC)) == 1:
                assert amla.amla_effective_splits(d) == 1 and amla.amla_workspace_bytes(d) == 0, (batch, blocks)


@pytest.mark.parametrize("heads,keys", [(16, 512), (40, 512), (32, 570), (128, 513)])
def test_values_beyond_fp16(exe, tmp_path, heads, keys):
    """Value columns of 1e5 and 1e-6 (no query looks at them) in tables of eight and nine blocks, no split factor given: every weight
    takes part in the sum that it is divided by, so the result is the column's value to FP32 rounding, half a BF16 step at most."""
    case = wl.make_case("range", 96, batch=1, s_q=1, heads=heads, seqlens=[keys])
    case.q_bits[..., :2] = 0
    bits = wl.f32_to_bf16_bits(np.array([1e5, 1e-6], np.float32))
    case.kv_bits[..., :2] = bits
    for variant in (MUL, ADD, COMP):
        out, _, splits = run_cpu(exe, tmp_path, case, variant)
        assert splits == 1 and np.all(np.abs(out[..., :2] / wl.bf16_bits_to_f32(bits) - 1) <= 2.0 ** -8), (variant, out[0, 0, 0, :2])


@pytest.mark.parametrize("rows", [33, 64, 96, 128, 256, 384, 512])
def test_fewer_balanced_workers_are_two_for_every_sequence(rows):
    """One workgroup per compute unit, or fewer on lower row tiles, but then at least two for every sequence."""
    s_q, heads = (rows // 128, 128) if rows % 128 == 0 else (1, rows)
    fewer = 0
    for batch in range(1, 65):
        for blocks in (4, 6, 7, 10, 16, 32, 47, 64, 125):
            workers = amla.amla_effective_splits(amla.make_desc(batch, s_q, heads, 20000, blocks, flags=amla.AMLA_FLAG_CAUSAL))
            most = min(256 // -(-rows // 128), batch * blocks)
            assert workers == most or 2 * batch <= workers < most
            fewer += workers < most
    assert fewer > 0
