"""amla_decode's arguments on their way through the native binding: what it refuses, with which error, before anything touches a GPU; and
that both built objects are asked for at import."""
import ctypes
import os
import shutil
import subprocess
import sys

import pytest

torch = pytest.importorskip("torch")
amla = pytest.importorskip("paper_2509_25224_amd.amla")


def test_host_tensors_and_other_objects_are_refused():
    q = torch.zeros(1, 1, 16, 576, dtype=torch.bfloat16)
    kv = torch.zeros(4, 64, 576, dtype=torch.bfloat16)
    table, lens = torch.zeros(1, 4, dtype=torch.int32), torch.zeros(1, dtype=torch.int32)
    with pytest.raises(ValueError, match="contiguous CUDA tensors"):
        amla.amla_decode(q, kv, table, lens, 0.1)
    with pytest.raises((TypeError, AttributeError)):
        amla.amla_decode(None, kv, table, lens, 0.1)
    with pytest.raises((TypeError, ValueError)):
        amla.amla_decode(q, kv, table, lens, 0.1, variant="add")


def test_the_first_argument_that_is_wrong_is_named():
    q = torch.zeros(1, 1, 16, 576, dtype=torch.bfloat16)
    kv = torch.zeros(4, 64, 576, dtype=torch.bfloat16)
    table, lens = torch.zeros(1, 4, dtype=torch.int32), torch.zeros(1, dtype=torch.int32)
    with pytest.raises(AttributeError, match="is_cuda"):
        amla.amla_decode(None, kv, table, lens, 0.1)
    with pytest.raises(ValueError, match="contiguous CUDA tensors"):
        amla.amla_decode(q, None, table, lens, 0.1)


@pytest.mark.parametrize("missing", ["libamla.so", "_amla_torch.so"])
def test_import_asks_for_both_objects(tmp_path, missing):
    package = os.path.dirname(os.path.abspath(amla.__file__))
    copy = tmp_path / "paper_2509_25224_amd"
    copy.mkdir()
    for name in ("__init__.py", "amla.py", "libamla.so", "_amla_torch.so"):
        if name != missing:
            shutil.copy(os.path.join(package, name), copy / name)
    run = subprocess.run([sys.executable, "-c", "import paper_2509_25224_amd.amla"], cwd=tmp_path, capture_output=True, text=True,
                         env=dict(os.environ, PYTHONPATH=str(tmp_path)))
    assert run.returncode != 0 and "ImportError" in run.stderr and missing + " is missing" in run.stderr


@pytest.mark.gpu
def test_what_device_calls_refuse_and_return():
    dev = torch.device("cuda:0")
    q = torch.zeros(2, 1, 16, 576, dtype=torch.bfloat16, device=dev)
    kv = torch.zeros(8, 64, 576, dtype=torch.bfloat16, device=dev)
    table, lens = torch.arange(8, dtype=torch.int32, device=dev).view(2, 4), torch.full((2,), 200, dtype=torch.int32, device=dev)
    bad = {"dtype": (q.float(), kv, table, lens), "strides": (q, kv.transpose(1, 2).contiguous().transpose(1, 2), table, lens),
           "dimensions": (q[0], kv, table, lens), "batch": (q, kv, table, lens[:1]), "widths": (q[..., :512].contiguous(), kv, table, lens)}
    for why, args in bad.items():
        with pytest.raises(ValueError):
            amla.amla_decode(*args, 0.1)
    with pytest.raises(IndexError):
        amla.amla_decode(q, kv, table.view(-1)[:2], lens, 0.1)
    for q_lens in (lens.long(), lens[:1], lens.view(1, 2), lens.cpu()):
        with pytest.raises(ValueError, match="q_lens"):
            amla.amla_decode(q, kv, table, lens, 0.1, q_lens=q_lens)
    for kw in ({"variant": 9}, {"flags": 4}, {"num_splits": 300}):
        with pytest.raises(amla.AmlaError):
            amla.amla_decode(q, kv, table, lens, 0.1, **kw)
    with pytest.raises(amla.AmlaError):
        amla.amla_decode(q, kv, table, lens, float("nan"))
    out, lse = torch.empty(2, 1, 16, 512, dtype=torch.bfloat16, device=dev), torch.empty(2, 1, 16, device=dev)
    got = amla.amla_decode(q, kv, table, lens, 0.1, out, lse, num_splits=2, workspace=torch.empty(1, dtype=torch.uint8, device=dev))
    assert got[0] is out and got[1] is lse
    assert amla.amla_decode(q, kv, table, lens, 0.1, want_lse=False)[1] is None
    again = amla.amla_decode(q, kv, table, lens, 0.1)
    assert again[0].shape == (2, 1, 16, 512) and again[0].dtype == torch.bfloat16 and again[1].dtype == torch.float32
    torch.cuda.synchronize()
    assert (lse - again[1]).abs().max() < 1e-5


@pytest.mark.gpu
def test_what_later_arguments_raise():
    dev = torch.device("cuda:0")
    q = torch.zeros(2, 1, 16, 576, dtype=torch.bfloat16, device=dev)
    kv = torch.zeros(8, 64, 576, dtype=torch.bfloat16, device=dev)
    table, lens = torch.arange(8, dtype=torch.int32, device=dev).view(2, 4), torch.full((2,), 200, dtype=torch.int32, device=dev)
    with pytest.raises(ctypes.ArgumentError):
        amla.amla_decode(q, kv, table, lens, "0.1")
    for kw in ({"q_lens": 3}, {"out": 3}, {"lse": 3}, {"workspace": 3}):
        with pytest.raises(AttributeError):
            amla.amla_decode(q, kv, table, lens, 0.1, **kw)
    with pytest.raises(RuntimeError, match="ambiguous"):   # no truth value
        amla.amla_decode(q, kv, table, lens, 0.1, want_lse=torch.zeros(2))
