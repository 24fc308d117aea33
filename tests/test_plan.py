"""The balanced decomposition's integer arithmetic (csrc/amla_plan.h), run on the host through the
C ABI (up to 256 workers, as many as a call can have, with the routines by which the kernels decide who owns which block;
above that in exact integers): plans by sequence.  Which workers meet a sequence the merge of the transposed family derives from these; what the
default family's workers note for theirs, and its plans by row tile, test_tile_plan_cpu.py reads."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from oracle import amla_oracle as orc
from paper_2509_25224_amd import amla


def _cases():
    rng = np.random.default_rng(7)
    yield [4096] * 64, 256
    yield [1, 63, 64, 65, 300, 1000], 8
    yield [0, 0, 5, 0], 3
    yield [70], 5                     # more workers than blocks
    yield [64 * 7] * 3, 7
    for _ in range(40):
        batch = int(rng.integers(1, 40))
        lens = rng.integers(0, 3000, batch)
        lens[rng.random(batch) < 0.15] = 0
        if lens.sum() == 0:
            lens[0] = 1
        yield lens.tolist(), int(rng.integers(1, 300))


@pytest.mark.parametrize("lens,workers", list(_cases()))
def test_pieces_tile_every_sequence_and_agree_with_the_combine_view(lens, workers):
    pieces, seq_workers = amla.amla_plan_segments(lens, workers)
    nb = [(n + 63) // 64 for n in lens]
    total = sum(nb)
    # every block of every sequence exactly once, pieces of a sequence in block order
    covered = {b: [] for b in range(len(lens))}
    for w, b, j0, j1, slot, full in pieces:
        assert 0 <= j0 < j1 <= nb[b]
        assert slot == w + b and 0 <= slot <= workers + len(lens) - 2
        covered[b].append((j0, j1, w, full))
    for b, runs in covered.items():
        at = 0
        for j0, j1, _, _ in runs:
            assert j0 == at
            at = j1
        assert at == nb[b]
        # a piece is full exactly when it is the sequence's only piece
        assert all(full == (len(runs) == 1) for _, _, _, full in runs)
        # what the transposed family's merge derives: first and last worker, and every worker in between
        # that owns any block has a piece of this sequence
        if nb[b] == 0:
            assert tuple(seq_workers[b]) == (-1, -1)
        else:
            ws = [w for _, _, w, _ in runs]
            assert ws == sorted(ws) and len(set(ws)) == len(ws)
            assert tuple(seq_workers[b]) == (ws[0], ws[-1])
            owning = [w for w in range(ws[0], ws[-1] + 1) if (w * total) // workers < ((w + 1) * total) // workers]
            assert owning == ws
    # slots are unique, pieces come in (worker, sequence) order, shares differ by at most one block
    slots = pieces[:, 4]
    assert np.all(np.diff(slots) > 0)
    share = np.zeros(workers, dtype=np.int64)
    for w, b, j0, j1, slot, full in pieces:
        share[w] += j1 - j0
    assert share.sum() == total and share.max() - share.min() <= 1


def test_merging_the_pieces_gives_the_definition():
    """The scheme itself, in fp64 on the CPU: attention over each piece's keys, merged per sequence
    with weights exp(lse_piece - lse) as the combine kernel does, equals attention over the whole
    sequence."""
    rng = np.random.default_rng(8)
    lens = [130, 0, 700, 64, 1500]
    workers = 6
    pieces, seq_workers = amla.amla_plan_segments(lens, workers)
    for b, n in enumerate(lens):
        if n == 0:
            continue
        Q = rng.standard_normal((4, 576))
        K = rng.standard_normal((n, 576))
        want, want_lse = orc.attention_rows(Q, K, 0.07)
        parts = []
        for w, pb, j0, j1, slot, full in pieces:
            if pb == b:
                parts.append(orc.attention_rows(Q, K[64 * j0:min(n, 64 * j1)], 0.07))
        lses = np.stack([l for _, l in parts])
        mx = lses.max(axis=0)
        wgt = np.exp(lses - mx)
        out = sum(o * w_[:, None] for (o, _), w_ in zip(parts, wgt)) / wgt.sum(axis=0)[:, None]
        assert np.abs(out - want).max() < 1e-12
        assert np.abs(mx + np.log(wgt.sum(axis=0)) - want_lse).max() < 1e-12


def test_plan_rejects_bad_arguments():
    with pytest.raises(amla.AmlaError):
        amla.amla_plan_segments([10, -1], 4)
    with pytest.raises(amla.AmlaError):
        amla.amla_plan_segments([10], 0)


CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2509_25224_amd", "csrc")


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    """The routines of amla_plan.h themselves, as the host compiler builds them."""
    tmp = tmp_path_factory.mktemp("plan")
    src = tmp / "plan.cpp"
    src.write_text(r'''
#include "amla_plan.h"
extern "C" int xcd_begin(int x, int w) { return plan_xcd_begin(x, w); }
// disagreements of the float and double forms with the integer ones, T blocks, 1 .. 256 workers: the first block of every
// worker, and the owner of the blocks around it
extern "C" long plan_mismatches(int64_t T) {
  long bad = 0;
  for (int64_t W = 1; W <= 256; ++W)
    for (int64_t w = 0; w <= W; ++w) {
      const int64_t first = plan_worker_begin(w, T, W);
      bad += (int64_t)plan_range_begin((uint32_t)w, (uint32_t)T, (uint32_t)W) != first;
      for (int64_t g = first - 1; g <= first + 1; ++g)
        if (g >= 0 && g < T)
          bad += (int64_t)plan_range_of_block((uint32_t)g, (uint32_t)T, (uint32_t)W) != plan_worker_of_block(g, T, W);
    }
  return bad;
}
''')
    subprocess.run(["g++", "-O2", "-shared", "-fPIC", "-I" + CSRC, "-o", str(tmp / "plan.so"), str(src)], check=True)
    return ctypes.CDLL(str(tmp / "plan.so"))


def test_workers_are_dealt_evenly_over_the_xcds(plan):
    for workers in range(1, 257):
        first = [plan.xcd_begin(x, workers) for x in range(9)]
        assert first[0] == 0 and first[8] == workers
        share = np.diff(first)
        assert share.min() == workers // 8 and share.max() == (workers + 7) // 8   # the grid has room for the latter


def test_the_kernels_arithmetic_is_exact(plan):
    """W <= 256 workers, T < 2^31 blocks: small totals, totals around multiples of the worker counts, the largest ones."""
    plan.plan_mismatches.restype, plan.plan_mismatches.argtypes = ctypes.c_long, [ctypes.c_int64]
    totals = set(range(1, 700)) | {2 ** k + d for k in range(10, 32) for d in (-2, -1, 0, 1)}
    totals |= {w * m + d for w in (3, 85, 127, 255, 256) for m in (77, 4099, (2 ** 31 - 2) // w) for d in (-1, 0, 1)}
    for total in sorted(t for t in totals if t < 2 ** 31):
        assert plan.plan_mismatches(total) == 0, total
