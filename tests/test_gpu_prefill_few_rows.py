"""Prefill products of a few prompt rows at their edges (needs an MI355X with
256 CUs: np = pairs / 256, rounded up, up to 32 pairs per workgroup): row counts
at both ends, every load layout, ragged last workgroups, K stages and slices,
and the first sizes past the rule, which take the tile products.  Each case is
held to the bounds of the prefill's oracle comparison: fp32 sums in another
order, and one bf16 rounding per cache entry."""
import pytest

from tests import test_gpu_probe as probe

pytestmark = pytest.mark.gpu

ONE = dict(n_layers=1)
I8 = dict(n_layers=1, wfmt="int8")
WIDE = dict(n_layers=1, n_heads=32, n_kv_heads=32, head_dim=128)

CASES = {
    # name: (config, cached rows before, prompt rows); gate/up's np in front
    "np1_rows11": (dict(ONE, ffn_dim=64), 0, 11),
    "np8_rows32": (dict(ONE, ffn_dim=2048), 0, 32),
    "np9_rows31": (dict(ONE, ffn_dim=2112), 5, 31),
    "np17_rows17": (dict(ONE, ffn_dim=4160), 0, 17),
    "np25_rows16": (dict(ONE, ffn_dim=6208), 3, 16),
    "np32_rows24": (dict(ONE, ffn_dim=8192), 0, 24),
    "np33_tiles": (dict(ONE, ffn_dim=8256), 0, 24),
    "rows33_tiles": (dict(ONE, ffn_dim=2048), 0, 33),
    "int8_np16": (dict(I8, ffn_dim=4096), 0, 32),
    "int8_np17": (dict(I8, ffn_dim=4160), 7, 23),
    "int8_np32": (dict(I8, ffn_dim=8192), 0, 12),
    # QKV np 24, ragged K stages (d 576), O split over K
    "qkv24": (dict(WIDE, d_model=576), 0, 23),
    "qkv24_int8": (dict(WIDE, d_model=576, wfmt="int8"), 2, 32),
    # QKV, O and down split over K; two layers
    "splits": (dict(d_model=2048, n_heads=16, n_kv_heads=8, head_dim=128, ffn_dim=4096), 0, 23),
    "splits_int8": (dict(d_model=2048, n_heads=32, n_kv_heads=8, ffn_dim=4096, wfmt="int8"), 0, 32),
    # odd head counts, d 320
    "ragged": (dict(d_model=320, ffn_dim=192, vocab=1000, n_heads=5, n_kv_heads=5), 0, 29),
    # a chunk of few rows behind a long one
    "behind_cache": (dict(ONE, ffn_dim=1024), 300, 20),
}


@pytest.mark.parametrize("name", list(CASES))
def test_prefill_few_rows(name, monkeypatch):
    kw, before, n = CASES[name]
    kw = dict(kw, prompt_len=before + n, n_steps=8)
    monkeypatch.setitem(probe.CASES, name, (kw, before, n))
    probe.test_prefill_matches_sequential_oracle(name)
