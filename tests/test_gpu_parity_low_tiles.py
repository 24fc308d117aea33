"""Row tiles of 16 and 32 rows for sequences of more rows (calls whose workgroups all run at once, cut by the library's own factor): the last
tile with one row, all but one and all of its rows, the calls on either side of a round of 256 workgroups, every decomposition."""
import numpy as np
import pytest

from test_gpu_parity import ADD, COMP, MUL, check, env, run_gpu, to_dev  # noqa: F401

pytestmark = pytest.mark.gpu
BALANCED, CAUSAL, ITER512 = 8, 16, 32


@pytest.mark.parametrize("lens", [[64, 0, 65, 128, 333], [700, 64, 0, 1300, 1024]])
@pytest.mark.parametrize("heads,s_q", [(33, 1), (47, 1), (48, 1), (128, 1), (43, 3), (128, 4)])
@pytest.mark.parametrize("variant,flags", [(ADD, 0), (MUL, 0), (COMP, 0), (ADD, ITER512), (MUL, BALANCED), (ADD, CAUSAL)])
def test_low_tiles(env, lens, heads, s_q, variant, flags):
    torch, orc, amla, wl = env
    case = wl.make_case("low", 101, batch=len(lens), s_q=s_q, heads=heads, seqlens=lens, spare_frac=0.2)
    q_lens = np.arange(len(lens), dtype=np.int32) % (s_q + 1) if flags & CAUSAL else None
    dev_q_lens = None if q_lens is None else torch.from_numpy(q_lens).cuda()
    out, lse = run_gpu(torch, amla, case, to_dev(torch, case), variant=variant, flags=flags, q_lens=dev_q_lens)
    want, want_lse = orc.decode(case.q_bits, case.kv_bits, case.block_table, case.seqlens, case.softmax_scale,
                                causal=bool(flags & CAUSAL), q_lens=q_lens)
    check(out, lse, want, want_lse, f"low tiles {heads} x {s_q} variant {variant} flags {flags}")


@pytest.mark.parametrize("batch", [16, 17, 32, 33, 64, 65])
def test_sides_of_a_round(env, batch):
    """Unsplit calls of 128 rows: tiles of 16 up to 32 sequences, of 32 up to 64, of 128 above, of 256 rows half as many."""
    torch, orc, amla, wl = env
    for s_q in (1, 2):
        case = wl.make_case("round", 102, batch=batch, s_q=s_q, heads=128, seqlens=[100 + 3 * b for b in range(batch)])
        out, lse = run_gpu(torch, amla, case, to_dev(torch, case), variant=ADD)
        want, want_lse = orc.decode(case.q_bits, case.kv_bits, case.block_table, case.seqlens, case.softmax_scale)
        # rows of 100 .. 300 keys reach outputs of 2 .. 4: half a BF16 step of the output, and the weights' rounding, 2^-9 relative each and
        # divided by the sum of the rounded ones, 2^-9 sum_k p_k |v_k - out| with a weighted mean distance below 3 for N(0, 1) values
        half_step = 2.0 ** (np.ceil(np.log2(np.maximum(np.abs(want), 2.0 ** -20))) - 9)
        assert np.all(np.abs(out - want) <= half_step + 3 * 2.0 ** -9) and np.abs(lse - want_lse).max() < 1e-4, (batch, s_q)


def tile_rows(amla, case, variant, flags):
    """Query rows of a workgroup under the library's own cut: the lowest tile whose workgroups all run at once, else 128."""
    own = amla.amla_effective_splits(amla.make_desc(case.batch, case.s_q, case.heads, case.num_blocks, case.max_blocks_per_seq, variant, 0, flags))
    rows, items = case.s_q * case.heads, own * (1 if flags & (BALANCED | CAUSAL) else case.batch)
    return next((t for t in (16, 32) if rows <= t or items * -(-rows // t) <= amla.amla_device_info()[0]), 128)


@pytest.mark.parametrize("heads,s_q", [(33, 1), (47, 1), (48, 1), (128, 1), (43, 3), (128, 4)])
@pytest.mark.parametrize("variant,flags", [(MUL, BALANCED), (ADD, CAUSAL), (COMP, CAUSAL)])
def test_balanced_calls_on_low_tiles(env, heads, s_q, variant, flags):
    """Balanced calls that test_low_tiles leaves on tiles of 128 rows, and the lower tile itself asserted."""
    torch, orc, amla, wl = env
    for lens in ([700, 64, 0, 1300, 1024], [3000]) if s_q == 4 else ([64, 0, 65, 128, 333], [1000, 0, 800]):
        case = wl.make_case("low", 101, batch=len(lens), s_q=s_q, heads=heads, seqlens=lens, spare_frac=0.2)
        assert tile_rows(amla, case, variant, flags) < 128
        q_lens = np.arange(len(lens), dtype=np.int32) % (s_q + 1) if flags & CAUSAL else None
        if q_lens is not None and len(lens) == 1:
            q_lens += 2   # (the one sequence: half of its tokens)
        dev_q_lens = None if q_lens is None else torch.from_numpy(q_lens).cuda()
        out, lse = run_gpu(torch, amla, case, to_dev(torch, case), variant=variant, flags=flags, q_lens=dev_q_lens)
        want, want_lse = orc.decode(case.q_bits, case.kv_bits, case.block_table, case.seqlens, case.softmax_scale,
                                    causal=bool(flags & CAUSAL), q_lens=q_lens)
        check(out, lse, want, want_lse, f"low tiles {heads} x {s_q} variant {variant} flags {flags} lens {lens}")


def test_which_tile_the_cases_above_run_on(env):
    _, _, amla, wl = env
    for lens in ([64, 0, 65, 128, 333], [700, 64, 0, 1300, 1024]):   # test_low_tiles without workers
        for heads, s_q in [(33, 1), (47, 1), (48, 1), (128, 1), (43, 3), (128, 4)]:
            for variant, flags in [(ADD, 0), (MUL, 0), (COMP, 0), (ADD, ITER512)]:
                assert tile_rows(amla, wl.make_case("low", 101, batch=5, s_q=s_q, heads=heads, seqlens=lens), variant, flags) < 128
    for batch in [16, 17, 32, 33, 64, 65]:   # test_sides_of_a_round
        for s_q in (1, 2):
            case = wl.make_case("round", 102, batch=batch, s_q=s_q, heads=128, seqlens=[100 + 3 * b for b in range(batch)])
            assert tile_rows(amla, case, ADD, 0) == (16 if batch * s_q <= 32 else 32 if batch * s_q <= 64 else 128)
