"""The merge of partial rows where its passes and row groups have remainders: more than 64 pieces of a sequence (a wave takes
64 at a time, where rows are so few that a workgroup merges each, all of them), more workers than blocks, row counts that no workgroup of four rows divides, more than 64
sequences in the plan's sums, empty sequences.  The bounds are the ones of test_gpu_parity.py."""
import numpy as np
import pytest

from test_gpu_parity import check, env, run_gpu, to_dev  # noqa: F401

pytestmark = pytest.mark.gpu
BALANCED, TRANSPOSED = 8, 128


@pytest.mark.parametrize("flags", [BALANCED, BALANCED | TRANSPOSED], ids=["fp16", "fp32"])
@pytest.mark.parametrize("heads,lens,workers", [(3, [9000], 130), (3, [4200], 200), (129, [4111, 70], 66),
                                                (5, [0] + [260 + 9 * i for i in range(70)] + [0], 256)])
def test_balanced_merge(env, flags, heads, lens, workers):
    torch, orc, amla, wl = env
    case = wl.make_case("merge", 81, batch=len(lens), s_q=1, heads=heads, seqlens=lens, spare_frac=0.1)
    out, lse = run_gpu(torch, amla, case, to_dev(torch, case), variant=1, num_splits=workers, flags=flags)
    want, want_lse = orc.decode(case.q_bits, case.kv_bits, case.block_table, case.seqlens, case.softmax_scale)
    check(out, lse, want, want_lse, f"merge heads {heads} workers {workers} flags {flags}")


@pytest.mark.parametrize("flags", [0, TRANSPOSED], ids=["fp16", "fp32"])
@pytest.mark.parametrize("heads,s_q,splits", [(3, 1, 100), (13, 1, 1), (21, 3, 9), (129, 1, 65), (128, 2, 8)])
def test_equal_share_merge_and_row_remainders(env, flags, heads, s_q, splits):
    torch, orc, amla, wl = env
    case = wl.make_case("merge", 82, batch=3, s_q=s_q, heads=heads, seqlens=[9000, 300, 0], spare_frac=0.1)
    out, lse = run_gpu(torch, amla, case, to_dev(torch, case), variant=1, num_splits=splits, flags=flags)
    want, want_lse = orc.decode(case.q_bits, case.kv_bits, case.block_table, case.seqlens, case.softmax_scale)
    check(out, lse, want, want_lse, f"merge heads {heads} s_q {s_q} splits {splits} flags {flags}")


@pytest.mark.parametrize("heads,s_q,lens,variant,flags",
                         [(128, 1, [9000] + [200, 0, 65] * 20, 1, 0), (128, 2, [6000, 300, 2000, 64, 900] * 5, 0, 32),
                          (16, 1, [16384, 128] * 30, 2, 0), (129, 1, [5000] + [0, 300] * 25, 1, 0),
                          (16, 1, [8192] * 95 + [8191], 1, 0), (128, 1, [3000, 0, 4096] * 3 + [0] * 55, 1, 0),
                          (128, 1, [1500, 0, 2048] * 3 + [0] * 55, 1, TRANSPOSED)])
def test_default_decomposition_of_ragged_batches(env, heads, s_q, lens, variant, flags):
    """No split factor given: bit for bit the call with the library's factor given (one batch: several rounds; the last two: mostly empty slots)."""
    torch, orc, amla, wl = env
    case = wl.make_case("ranges", 84, batch=len(lens), s_q=s_q, heads=heads, seqlens=lens, spare_frac=0.05)
    out, lse = run_gpu(torch, amla, case, to_dev(torch, case), variant=variant, flags=flags)
    want, want_lse = orc.decode(case.q_bits, case.kv_bits, case.block_table, case.seqlens, case.softmax_scale)
    check(out, lse, want, want_lse, f"ranges heads {heads} s_q {s_q}")
    splits = amla.amla_effective_splits(amla.make_desc(case.batch, s_q, heads, case.num_blocks, case.max_blocks_per_seq,
                                                       variant, 0, flags))
    assert splits > 1
    same, same_lse = run_gpu(torch, amla, case, to_dev(torch, case), variant=variant, num_splits=splits, flags=flags)
    assert np.array_equal(out, same) and np.array_equal(lse, same_lse)


@pytest.mark.parametrize("heads,lens,splits,flags", [(128, [64, 0] + [64] * 6 + [30 * 64], 65, 0), (1100, [128, 300], 129, 0),
                                                     (128, [64, 300], 65, TRANSPOSED), (43, [192], 193, TRANSPOSED)])
def test_first_64_shares_without_blocks(env, heads, lens, splits, flags):
    """Sequences of one, two and three blocks in so many shares that the first 64, what a wave merges at a time, hold nothing."""
    torch, orc, amla, wl = env
    case = wl.make_case("late_shares", 95, batch=len(lens), s_q=1, heads=heads, seqlens=lens, spare_frac=0.1)
    out, lse = run_gpu(torch, amla, case, to_dev(torch, case), variant=1, num_splits=splits, flags=flags)
    want, want_lse = orc.decode(case.q_bits, case.kv_bits, case.block_table, case.seqlens, case.softmax_scale)
    check(out, lse, want, want_lse, f"late shares heads {heads} splits {splits} flags {flags}")


@pytest.mark.parametrize("heads,lens,pieces,flags", [(128, [70 * 64 - 3] + [300] * 8, 65, 0), (48, [9000] + [0] * 9, 256, BALANCED),
                                                     (48, [200 * 64] + [0] * 9, 200, BALANCED)])
def test_wave_merge_of_fp16_rows_in_several_passes(env, heads, lens, pieces, flags):
    """So many rows that a wave merges each of them: 65 pieces, 141 of 256 workers (passes with gaps), 200."""
    torch, orc, amla, wl = env
    case = wl.make_case("passes", 98, batch=len(lens), s_q=1, heads=heads, seqlens=lens, spare_frac=0.1)
    assert len(lens) * heads > 16 * -(-pieces // (len(lens) if flags else 1))
    out, lse = run_gpu(torch, amla, case, to_dev(torch, case), variant=1, num_splits=pieces, flags=flags)
    want, want_lse = orc.decode(case.q_bits, case.kv_bits, case.block_table, case.seqlens, case.softmax_scale)
    check(out, lse, want, want_lse, f"passes heads {heads} pieces {pieces} flags {flags}")
