"""The prefill products' tile shapes and K splits at their edges (needs an
MI355X): row counts one past a tile, an odd number of 128-row units, splits
into 2, 4 and 8 slices, each at the smallest model whose cost picks that shape.
The last entry of a case is what it takes (tests/test_prefill_plan.py holds the
library to it): shape B(ig) / W(ide) / S(hort) and K slices of QKV, O, gate/up
and down.  Each case is held to the bounds of the prefill's oracle comparison:
fp32 sums in another order, and one bf16 rounding per cache entry."""
import pytest

from tests import test_gpu_probe as probe

pytestmark = pytest.mark.gpu

WIDE_D = dict(d_model=1024, ffn_dim=4096, n_heads=8, n_kv_heads=8, head_dim=128)

CASES = {
    # gate/up: 255 units (the last tile's second unit lies past the end) and one
    # live row in the second row tile
    "big_odd_units": (dict(n_layers=1, ffn_dim=16320), 0, 129, "S1 S1 B1 S8"),
    # gate/up: the third prompt block starts at the last row
    "wide_split2": (dict(n_layers=1, d_model=1024, n_heads=16, n_kv_heads=16, ffn_dim=16384),
                    0, 33, "S4 S4 W2 S8"),
    "wide_split4": (dict(n_layers=1, d_model=2048, n_heads=32, n_kv_heads=8, ffn_dim=8192), 0, 33,
                    "S4 S4 W4 S8"),
    "big_split2": (dict(n_layers=1, d_model=2048, n_heads=32, n_kv_heads=8, ffn_dim=16384), 0, 65,
                   "S2 S4 B2 S8"),
    # QKV and O in 9 row tiles of 64, the last of 8 rows, behind a cache
    "wide_qkv_o_split2": (dict(n_layers=1, d_model=2048, n_heads=32, n_kv_heads=8, ffn_dim=64),
                          5, 520, "W2 W2 S4 W1"),
    # QKV and O in 6 row tiles of 128, the last of 60 rows
    "big_o_split2": (dict(n_layers=1, d_model=4096, n_heads=64, n_kv_heads=16, ffn_dim=64), 0, 700,
                     "B1 B2 S8 W1"),
    # down has two stages of K
    "big_all": (dict(n_layers=1, d_model=4096, n_heads=32, n_kv_heads=8, head_dim=128, ffn_dim=64),
                0, 1030, "B1 B1 S4 B1"),
    # two layers, int8
    "int8_mixed": (dict(WIDE_D, wfmt="int8"), 0, 700, "W1 S1 B1 S4"),
    # QKV: a last row tile of 92 rows
    "int8_big_wide": (dict(WIDE_D, wfmt="int8", n_layers=1), 0, 1500, "B1 S1 W1 W2"),
}


@pytest.mark.parametrize("name", list(CASES))
def test_prefill_tile_shapes(name, monkeypatch):
    kw, before, n, _ = CASES[name]
    kw = dict(kw, prompt_len=before + n, n_steps=8)
    monkeypatch.setitem(probe.CASES, name, (kw, before, n))
    probe.test_prefill_matches_sequential_oracle(name)
