"""Row tiles of 16 and 32 rows under per-sequence token counts in the CPU build (see test_cpu_build.py): a tile of padding tokens alone is
not worked, that is, none of its sequence's cache blocks is loaded for it, and its rows come back as zeros."""
import numpy as np
import pytest

from paper_2509_25224_amd import workloads as wl
from test_cpu_build import ADD, BALANCED, CAUSAL, COMP, MUL, check, exe, launch_info, run_cpu  # noqa: F401

LOADS_OF_A_BLOCK = 64 * 72   # 16-byte loads


@pytest.mark.parametrize("heads,columns,tile_rows,variant,flags", [(16, 5, 16, ADD, CAUSAL), (24, 5, 16, COMP, BALANCED),
                                                                   (16, 40, 32, MUL, CAUSAL), (20, 40, 32, ADD, BALANCED)])
def test_low_tiles_of_padding_tokens(exe, tmp_path, heads, columns, tile_rows, variant, flags):
    lens, q_lens = [60, 300, 130, 64], [2, 1, 4, 0]
    batch = 2 if columns == 40 else 4
    for first in range(0, 4, batch):   # a sequence in one piece, in several, without tokens
        part, tokens = lens[first:first + batch], q_lens[first:first + batch]
        case = wl.make_case("low_padding", 106, batch=batch, s_q=4, heads=heads, seqlens=part, max_blocks_per_seq=columns, spare_frac=0.2)
        out, lse, _ = run_cpu(exe, tmp_path, case, variant, flags=flags, q_lens=tokens)
        check(out, lse, case, causal=flags == CAUSAL, q_lens=tokens)
        tiles, _, loads, _ = launch_info(tmp_path)
        assert tiles == -(-4 * heads // tile_rows)
        assert loads == LOADS_OF_A_BLOCK * sum(-(-n // 64) * -(-t * heads // tile_rows) for n, t in zip(part, tokens))
