"""The kernels of 128 query rows in the CPU build (see test_cpu_build.py), the tile asserted as launched: the library's own cut of
calls this small goes to tiles of 16 and 32, so the factors here are others, or the table is wide enough for another cut."""
import copy

import numpy as np
import pytest

from paper_2509_25224_amd import workloads as wl
from test_cpu_build import ADD, BALANCED, CAUSAL, COMP, ITER512, MUL, NO_SKIP, check, exe, launch_info, run_cpu  # noqa: F401


def ragged(seed):
    # 160 rows: two tiles, the second with 32 rows; a table of 24 columns, which the library would cut
    return wl.make_case("edges", seed, batch=7, s_q=2, heads=80, seqlens=[1, 63, 0, 64, 65, 200, 330], spare_frac=0.25, max_blocks_per_seq=24)


@pytest.mark.parametrize("variant,flags,ns", [(MUL, 0, 1), (ADD, 0, 1), (COMP, 0, 1), (MUL, 0, 3), (ADD, 0, 3), (COMP, 0, 2), (COMP, 0, 3),
                                              (ADD, ITER512, 3), (MUL, ITER512, 1)])
def test_ragged_splits(exe, tmp_path, variant, flags, ns):
    case = ragged(51)
    out, lse, splits = run_cpu(exe, tmp_path, case, variant, flags=flags, ns=ns)
    assert splits == ns and next(launch_info(tmp_path)) == 2
    check(out, lse, case)
    assert np.all(out[2] == 0) and np.all(np.isneginf(lse[2]))


@pytest.mark.parametrize("variant", [MUL, ADD, COMP])
def test_wide_logits_and_slots_past_the_end(exe, tmp_path, variant):
    wide = wl.make_case("wide_row", 72, batch=1, s_q=1, heads=40, seqlens=[700], q_sigma=6.0)
    a = run_cpu(exe, tmp_path, wide, variant, ns=1)
    assert next(launch_info(tmp_path)) == 1   # (the library would cut it, on lower tiles)
    check(a[0], a[1], wide, peaked=True)
    b = run_cpu(exe, tmp_path, wide, variant, flags=NO_SKIP, ns=1)
    check(b[0], b[1], wide, peaked=True)
    if variant == ADD:
        assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
    dirty = copy.copy(wide)
    dirty.kv_bits = wide.kv_bits.copy()
    dirty.kv_bits[int(wide.block_table[0, 700 // 64]), 700 % 64:, :] = 0x7FC0   # NaN in every slot past the end of the last block
    c = run_cpu(exe, tmp_path, dirty, variant, ns=1)
    assert np.array_equal(a[0], c[0]) and np.array_equal(a[1], c[1])


@pytest.mark.parametrize("variant", [MUL, ADD])
@pytest.mark.parametrize("flags,ns", [(0, 1), (0, 3), (BALANCED, 5), (CAUSAL, 0)])
def test_iteration_of_512_keys_on_128_rows(exe, tmp_path, variant, flags, ns):
    case = wl.make_case("it512", 81, batch=4, s_q=2, heads=40, seqlens=[1500, 570, 512, 448], spare_frac=0.25)
    out, lse, _ = run_cpu(exe, tmp_path, case, variant, flags=ITER512 | flags, ns=ns)
    assert next(launch_info(tmp_path)) == 1
    check(out, lse, case, causal=bool(flags & CAUSAL))
