"""The default entry (no split factor given): a call is cut by its shape alone, so that a sequence's bits are those of the
call with the same factor given explicitly and do not move with its neighbours' lengths.  The library's source compiled
for the host (see test_cpu_build.py), under AddressSanitizer with a workspace of exactly the documented size."""
import numpy as np
import pytest

from paper_2509_25224_amd import workloads as wl
from test_cpu_build import check, exe, run_cpu  # noqa: F401

LONG_AND_EMPTY = [0] * 20 + [5000] + [40, 0] * 9 + [64, 65, 129] + [0] * 18   # one long sequence between short and empty ones


def _case(heads, s_q, lens, columns=0):
    """`columns`: a block table laid out for longer sequences (the library splits by it)."""
    case = wl.make_case("default", 83, batch=len(lens), s_q=s_q, heads=heads, seqlens=lens, spare_frac=0.1)
    if columns > case.max_blocks_per_seq:
        wide = np.full((case.batch, columns), -1, np.int32)
        wide[:, :case.max_blocks_per_seq] = case.block_table
        case.block_table = wide
    return case


@pytest.mark.parametrize("heads,s_q,lens,columns,variant,flags,static",
                         [(16, 1, LONG_AND_EMPTY, 0, 1, 0, False), (3, 1, LONG_AND_EMPTY, 0, 0, 32, True),
                          (129, 1, [5000] + [0, 63] * 15, 0, 2, 0, False), (16, 1, [700, 500], 600, 1, 0, False),
                          (16, 1, [600, 0, 520], 0, 1, 0, False), (130, 1, [700, 0, 65], 200, 0, 0, True)])
def test_default_is_the_explicit_split(exe, tmp_path, heads, s_q, lens, columns, variant, flags, static):
    case = _case(heads, s_q, lens, columns)
    out, lse, splits = run_cpu(exe, tmp_path, case, variant, flags=flags, static_ws=static)
    assert splits > 1
    want, want_lse, _ = run_cpu(exe, tmp_path, case, variant, flags=flags, ns=splits)
    assert np.array_equal(out, want) and np.array_equal(lse, want_lse)
    check(out, lse, case)


def test_a_sequence_does_not_depend_on_its_neighbours_lengths(exe, tmp_path):
    case = _case(16, 1, [900, 5000] + [40, 0] * 29)
    out, lse, splits = run_cpu(exe, tmp_path, case, 1)
    assert splits > 1
    case.seqlens = case.seqlens.copy()
    case.seqlens[1] = 1000
    alone, alone_lse, same_splits = run_cpu(exe, tmp_path, case, 1)
    assert same_splits == splits
    keep = np.arange(case.batch) != 1
    assert np.array_equal(out[keep], alone[keep]) and np.array_equal(lse[keep], alone_lse[keep])


def test_more_pieces_than_a_wave_merge_to_the_same_bits(exe, tmp_path):
    """50 blocks in 50 shares of one, and in 100 shares of which 50 are empty: the same pieces, so the same merge, also
    where it takes more than one pass over the pieces (FP32 rows; the FP16 rows of so few go to the workgroup-per-row merge)."""
    case = _case(24, 1, [50 * 64 - 7, 50 * 64])
    for flags in (0, 128):   # FP16 and FP32 partial rows
        out, lse, _ = run_cpu(exe, tmp_path, case, 1, flags=flags, ns=100)
        want, want_lse, _ = run_cpu(exe, tmp_path, case, 1, flags=flags, ns=50)
        assert np.array_equal(out, want) and np.array_equal(lse, want_lse)
        check(out, lse, case)


@pytest.mark.parametrize("heads,lens,flags,ns", [(1100, [4200], 0, 66), (35, [70 * 64 - 1] + [0] * 9, 8, 200)])
def test_wave_merge_of_fp16_rows_in_several_passes(exe, tmp_path, heads, lens, flags, ns):
    """So many rows that a wave merges each of them, 64 pieces at a time: 66 pieces, and 70 of 200 workers (four passes with gaps)."""
    case = wl.make_case("passes", 97, batch=len(lens), s_q=1, heads=heads, seqlens=lens)
    assert len(lens) * heads > 16 * -(-ns // (len(lens) if flags else 1))
    out, lse, _ = run_cpu(exe, tmp_path, case, 1, flags=flags, ns=ns)
    check(out, lse, case)


@pytest.mark.parametrize("variant", [0, 1, 2])
def test_rows_past_the_end_count_as_the_sequences_first(exe, tmp_path, variant):
    """A wave's 32 rows share the decision to keep the reference: 24 rows give the bits of 32 rows whose last eight repeat
    row 0.  (The last row is zero but for eight large values in its second half: rows made of those would decide otherwise.)"""
    lens = [700, 640, 500, 65, 900, 1000]
    short = wl.make_case("rows", 85, batch=6, s_q=1, heads=24, seqlens=lens)
    full = wl.make_case("rows", 85, batch=6, s_q=1, heads=32, seqlens=lens)
    full.kv_bits, full.block_table = short.kv_bits, short.block_table
    last = np.zeros(576, np.float32)
    last[288:296] = 32
    short.q_bits[:, :, 23] = wl.f32_to_bf16_bits(last)
    full.q_bits = np.concatenate([short.q_bits, np.repeat(short.q_bits[:, :, :1], 8, axis=2)], axis=2)
    out, lse, _ = run_cpu(exe, tmp_path, short, variant, ns=1)
    want, want_lse, _ = run_cpu(exe, tmp_path, full, variant, ns=1)
    assert np.array_equal(out, want[:, :, :24]) and np.array_equal(lse, want_lse[:, :, :24])
