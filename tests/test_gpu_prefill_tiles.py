"""The prefill products' tile shapes and K splits at their edges (needs an
MI355X): row counts one past a tile, an odd number of 128-row units, splits
into 2, 4 and 8 slices, each at the smallest model whose cost picks that shape
(in the comments: product, shape B(ig) / W(ide) / S(hort), K slices).  Each
case is held to the bounds of the prefill's oracle comparison: fp32 sums in
another order, and one bf16 rounding per cache entry."""
import pytest

import synth
from tests import test_gpu_probe as probe

pytestmark = pytest.mark.gpu

WIDE_D = dict(d_model=1024, ffn_dim=4096, n_heads=8, n_kv_heads=8, head_dim=128)

CASES = {
    # gate/up B1 with 255 units (the last tile's second unit lies past the
    # end) and one live row in the second row tile; down S8
    "big_odd_units": (dict(n_layers=1, ffn_dim=16320), 0, 129),
    # gate/up W2: the third prompt block starts at the last row
    "wide_split2": (dict(n_layers=1, d_model=1024, n_heads=16, n_kv_heads=16, ffn_dim=16384),
                    0, 33),
    "wide_split4": (dict(n_layers=1, d_model=2048, n_heads=32, n_kv_heads=8, ffn_dim=8192), 0, 33),
    "big_split2": (dict(n_layers=1, d_model=2048, n_heads=32, n_kv_heads=8, ffn_dim=16384), 0, 65),
    # QKV and O W2 in 9 row tiles of 64, the last of 8 rows, behind a cache
    "wide_qkv_o_split2": (dict(n_layers=1, d_model=2048, n_heads=32, n_kv_heads=8, ffn_dim=64),
                          5, 520),
    # QKV B1, O B2 in 6 row tiles of 128, the last of 60 rows
    "big_o_split2": (dict(n_layers=1, d_model=4096, n_heads=64, n_kv_heads=16, ffn_dim=64), 0, 700),
    # QKV, O and down B1; down has two stages of K
    "big_all": (dict(n_layers=1, d_model=4096, n_heads=32, n_kv_heads=8, head_dim=128, ffn_dim=64),
                0, 1030),
    # two layers, int8: QKV W1, O S1, gate/up B1, down S4
    "int8_mixed": (dict(WIDE_D, wfmt="int8"), 0, 700),
    # QKV B1 with a last row tile of 92 rows, gate/up W1, down W2
    "int8_big_wide": (dict(WIDE_D, wfmt="int8", n_layers=1), 0, 1500),
}


@pytest.mark.parametrize("name", list(CASES))
def test_prefill_tile_shapes(name, monkeypatch):
    kw, before, n = CASES[name]
    kw = dict(kw, prompt_len=before + n, n_steps=8)
    monkeypatch.setitem(probe.CASES, name, (kw, before, n))
    probe.test_prefill_matches_sequential_oracle(name)
