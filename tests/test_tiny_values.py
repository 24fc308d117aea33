"""ADD_COMP over value columns of 2^-112 whose accumulator has to lose more exponent than it has: an uncut call has BF16's range, so
what a first block left there must end as zero and not stay 2^30 times too large beside the block that carries the weight."""
import numpy as np
import pytest

from paper_2509_25224_amd import workloads as wl
from test_cpu_build import BALANCED, COMP, exe, run_cpu  # noqa: F401
from test_gpu_parity import env, run_gpu, to_dev  # noqa: F401

TINY = 2.0 ** -112
# 40 rows in the general kernel (one worker, which is not the library's own number) and on low row tiles, 16 rows
CALLS = [(40, BALANCED, 1), (40, 0, 0), (16, 0, 0)]


def _case(heads):
    """Keys of one weight, but for the 65th, 33 base-2 units above them: its value row is the result to 2^-26."""
    case = wl.make_case("tiny_values", 105, batch=1, s_q=1, heads=heads, seqlens=[128], table="identity", softmax_scale=float(np.log(2)))
    case.q_bits[...] = 0
    case.q_bits[..., 575] = wl.f32_to_bf16_bits(np.full(1, 33, np.float32))
    case.kv_bits[..., 575] = 0
    case.kv_bits[1, 0, 575:] = wl.f32_to_bf16_bits(np.ones(1, np.float32))
    case.kv_bits[..., 3], case.kv_bits[..., 5] = wl.f32_to_bf16_bits(np.array([TINY, -TINY], np.float32))
    return case


def _check(out, case):
    assert np.all(np.abs(out[..., [3, 5]] / [TINY, -TINY] - 1) <= 2.0 ** -8), out[0, 0, 0, [3, 5]] / TINY
    row = wl.bf16_bits_to_f32(case.kv_bits[1, 0, :512])
    assert np.all(np.abs(out - row) <= np.abs(row) * 2.0 ** -8 + 2.0 ** -20)


@pytest.mark.parametrize("heads,flags,ns", CALLS)
def test_tiny_value_columns(exe, tmp_path, heads, flags, ns):
    case = _case(heads)
    out, _, _ = run_cpu(exe, tmp_path, case, COMP, flags=flags, ns=ns)
    _check(out, case)


@pytest.mark.gpu
@pytest.mark.parametrize("heads,flags,ns", CALLS)
def test_tiny_value_columns_on_the_gpu(env, heads, flags, ns):
    torch, orc, amla, _ = env
    case = _case(heads)
    out, _ = run_gpu(torch, amla, case, to_dev(torch, case), variant=COMP, flags=flags, num_splits=ns)
    _check(out, case)
