"""Per-sequence token counts in the CPU build (see test_cpu_build.py): the balanced plan goes by row tiles where a quarter of the (tile, block) pairs are
padding and that makes the workers' ranges enough shorter, else by sequences; the workspace of exactly the documented size holds either one's pieces
and notes."""
import numpy as np
import pytest

from paper_2509_25224_amd import workloads as wl
from test_cpu_build import ADD, BALANCED, CAUSAL, COMP, MUL, check, exe, launch_info, run_cpu  # noqa: F401


@pytest.mark.parametrize("heads,s_q,lens,q_lens,workers,variant,flags,static", [
    (65, 2, [700, 0, 520, 580], [1, 2, 2, 0], 1, ADD, CAUSAL, False),      # two tiles, the last of two rows; one worker a tile, one empty sequence
    (65, 2, [700, 0, 520, 580], [1, 2, 2, 0], 40, MUL, CAUSAL, True),      # more workers than units
    (129, 1, [1200, 513], [0, 1], 3, COMP, BALANCED, False),               # a tile of one row; a sequence of many keys without tokens
    (128, 2, [512, 511], [1, 2], 2, ADD, CAUSAL, False),                   # 24 of 32 pairs
    (128, 2, [576, 512], [2, 1], 2, ADD, CAUSAL, False),                   # 26 of 34
    (128, 2, [512, 448], [1, 1], 2, ADD, CAUSAL, False),                   # half of them
    (129, 1, [600], [1], 1, MUL, BALANCED, False)])                        # the smallest workspace of two tiles: two slots' worth
def test_plans_by_tile_and_by_sequence(exe, tmp_path, heads, s_q, lens, q_lens, workers, variant, flags, static):
    case = wl.make_case("tile_plan", 103, batch=len(lens), s_q=s_q, heads=heads, seqlens=lens, spare_frac=0.2)
    out, lse, _ = run_cpu(exe, tmp_path, case, variant, flags=flags, ns=workers, q_lens=q_lens, static_ws=static)
    check(out, lse, case, causal=bool(flags & CAUSAL), q_lens=q_lens)
    for b, k in enumerate(q_lens):
        assert np.all(out[b, k:] == 0) and np.all(np.isneginf(lse[b, k:]))


@pytest.mark.parametrize("heads,s_q,lens,q_lens,workers,variant,flags,static,by_tile", [
    (65, 2, [700, 64, 1000, 580], [1, 2, 2, 0], 2, ADD, CAUSAL, False, True),     # two tiles, the last of two rows
    (65, 2, [700, 64, 1000, 580], [1, 2, 2, 0], 1, ADD, CAUSAL, False, False),    # a workspace with slots for one worker by tile
    (65, 2, [700, 64, 1000, 580], [1, 2, 2, 0], 40, MUL, CAUSAL, True, False),    # more workers than units
    (65, 2, [700, 0, 520, 580], [1, 2, 2, 0], 1, COMP, CAUSAL, False, True),      # one of them empty
    (129, 1, [1200, 513], [0, 1], 3, COMP, BALANCED, False, True),                # a tile of one row; a sequence of many keys without tokens
    (128, 2, [512, 511], [1, 2], 2, ADD, CAUSAL, False, True),                    # 24 of 32 pairs
    (128, 2, [512, 511], [1, 2], 6, ADD, CAUSAL, True, True),                     # two units for 2.67 blocks, one piece more
    (128, 2, [512, 511], [1, 2], 7, MUL, CAUSAL, False, False),                   # 1.71 for 2.29, 1.17 more
    (128, 2, [576, 512], [2, 1], 2, ADD, CAUSAL, False, False),                   # 26 of 34 pairs
    (128, 2, [512, 448], [1, 1], 2, ADD, CAUSAL, False, True),                    # half of them
    (129, 1, [600], [1], 1, MUL, BALANCED, False, False)])                        # the smallest workspace of two tiles: two slots' worth
def test_which_plan_is_taken(exe, tmp_path, heads, s_q, lens, q_lens, workers, variant, flags, static, by_tile):
    case = wl.make_case("tile_plan", 103, batch=len(lens), s_q=s_q, heads=heads, seqlens=lens, spare_frac=0.2)
    out, lse, _ = run_cpu(exe, tmp_path, case, variant, flags=flags, ns=workers, q_lens=q_lens, static_ws=static)
    check(out, lse, case, causal=bool(flags & CAUSAL), q_lens=q_lens)
    tiles, went_by_tile, _, _ = launch_info(tmp_path)
    assert tiles == 2 and went_by_tile == by_tile
    for b, k in enumerate(q_lens):
        assert np.all(out[b, k:] == 0) and np.all(np.isneginf(lse[b, k:]))


@pytest.mark.parametrize("heads,lens,workers,variant", [(20, [200, 0, 64, 330], 23, ADD), (130, [64, 700], 200, MUL), (2, [900], 256, COMP)])
def test_workers_are_numbered_without_gaps(exe, tmp_path, heads, lens, workers, variant):
    """More workers than blocks: a block each for as many as there are blocks, and those of a sequence side by side for the merge."""
    case = wl.make_case("no_gaps", 109, batch=len(lens), s_q=1, heads=heads, seqlens=lens, spare_frac=0.2)
    out, lse, _ = run_cpu(exe, tmp_path, case, variant, flags=BALANCED, ns=workers)
    check(out, lse, case)
    tiles, by_tile, _, _ = launch_info(tmp_path)
    notes = np.fromfile(str(tmp_path / "out.bin.info"), np.int32, offset=32).reshape(len(lens), tiles, 2)
    before = 0
    for b, n in enumerate(lens):
        blocks = -(-n // 64)
        assert not by_tile and (blocks == 0 or np.all(notes[b] == [before, before + blocks - 1]))
        before += blocks


@pytest.mark.parametrize("heads,s_q,lens,q_lens,columns,tile_rows,variant,flags,static,by_tile", [
    (32, 16, [20 * 64 - 3], [1], 32, 16, ADD, CAUSAL, False, True),               # 8 workers by sequence: 2.5 blocks each, or 40 units for 256
    (32, 16, [12 * 64], [1], 32, 16, MUL, CAUSAL, True, False),                   # 1.5 blocks less 24 / 256 of a unit
    (32, 12, [25 * 64, 20 * 64 - 1], [1, 2], 47, 32, COMP, BALANCED, True, True),   # 21 workers by sequence, 252 by tile
    (33, 12, [1500, 0, 1000], [2, 5, 0], 32, 16, MUL, CAUSAL, False, True),       # tokens that share tiles; the last tile of twelve rows
    (33, 12, [700, 0, 300], [2, 5, 1], 32, 16, ADD, CAUSAL, False, False)])
def test_plans_on_low_tiles(exe, tmp_path, heads, s_q, lens, q_lens, columns, tile_rows, variant, flags, static, by_tile):
    """The library's own number of workers, on lower tiles: by row tile where that makes ranges shorter by a block and a half."""
    case = wl.make_case("low_tile_plan", 110, batch=len(lens), s_q=s_q, heads=heads, seqlens=lens, spare_frac=0.2, max_blocks_per_seq=columns)
    out, lse, _ = run_cpu(exe, tmp_path, case, variant, flags=flags, q_lens=q_lens, static_ws=static)
    check(out, lse, case, causal=bool(flags & CAUSAL), q_lens=q_lens)
    tiles, went_by_tile, _, _ = launch_info(tmp_path)
    assert tiles == -(-s_q * heads // tile_rows) and went_by_tile == by_tile
    for b, k in enumerate(q_lens):
        assert np.all(out[b, k:] == 0) and np.all(np.isneginf(lse[b, k:]))
