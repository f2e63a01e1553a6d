"""Which kernel, K split and row pairs each product of a prefill takes on 256 CUs
(host): the GPU cases of the tile shapes and of the few-row products are the ones
they are meant to be, and so are the workloads'."""
import ctypes

import pytest

import synth
from paper_2604_09752_amd import binding as B
from tests import test_gpu_prefill_few_rows as few
from tests import test_gpu_prefill_tiles as tiles
from tests import test_gpu_probe as probe


def plan(cfg, rows, cus=256):
    """Kernel and K slices (/ row pairs) of QKV, O, gate/up and down."""
    out = (ctypes.c_int32 * 12)()
    assert B.lib().aio_prefill_plan(ctypes.byref(B.make_config(cfg)), rows, cus, out) == B.AIO_OK
    return " ".join("%s%d%s" % ("BWSF"[out[i]], out[i + 1], "/%d" % out[i + 2] if out[i + 2] else "")
                    for i in range(0, 12, 3))


@pytest.mark.parametrize("name", list(tiles.CASES))
def test_tile_cases(name):
    kw, before, n, want = tiles.CASES[name]
    assert plan(probe.TINY.with_(name=name, **dict(kw, prompt_len=before + n, n_steps=8)), n) == want


@pytest.mark.parametrize("name", list(few.CASES))
def test_few_row_cases(name):
    kw, before, n, want = few.CASES[name]
    assert plan(probe.TINY.with_(name=name, **dict(kw, prompt_len=before + n, n_steps=8)), n) == want


@pytest.mark.parametrize("name,want", [("split_k", "F2/12 F2 F2/32 F8"),
                                       ("split_k_int8", "S2 S4 S1 S8"),
                                       ("wide_tiles", "W1 S1 W1 W2"), ("n2048", "W1 S1 W1 S2")])
def test_probe_cases(name, want):
    kw, _, n = probe.CASES[name]
    assert plan(probe.TINY.with_(name=name, **kw), n) == want


@pytest.mark.parametrize("model,rows,want", [
    ("1b", 23, "F4/32 F4 F1/22 F8"), ("1b", 33, "S4 S4 W4 S8"), ("1b", 389, "W2 S1 B1 W4"),
    ("1b", 2048, "B1 W1 B1 B2"), ("7b", 23, "F1/24 F4 S4 F4"), ("7b", 32, "S4 F4 S4 F4"),
    ("7b", 1000, "B2 B2 B1 B2")])
def test_workloads(model, rows, want):
    assert plan(synth.CONFIGS[model], rows) == want


def test_rejects():
    c, out = ctypes.byref(B.make_config(synth.CONFIGS["1b"])), (ctypes.c_int32 * 12)()
    f = B.lib().aio_prefill_plan
    assert f(c, 0, 256, out) == B.AIO_EINVAL
    assert f(c, 8, 0, out) == B.AIO_EINVAL
    assert f(c, 8, 256, None) == B.AIO_EINVAL
    assert f(None, 8, 256, out) == B.AIO_EINVAL
