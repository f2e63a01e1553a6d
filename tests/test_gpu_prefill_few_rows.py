"""Prefill products of a few prompt rows at their edges (needs an MI355X with
256 CUs: np = pairs / 256, rounded up, up to 32 pairs per workgroup): row counts
at both ends, every load layout, ragged last workgroups, K stages and slices,
and the first sizes past the rule, which take the tile products (the plans are
held to by tests/test_prefill_plan.py).  Each case is held to the bounds of the prefill's oracle comparison: fp32 sums in another
order, and one bf16 rounding per cache entry."""
import pytest

from tests import test_gpu_probe as probe

pytestmark = pytest.mark.gpu

ONE = dict(n_layers=1)
I8 = dict(n_layers=1, wfmt="int8")
WIDE = dict(n_layers=1, n_heads=32, n_kv_heads=32, head_dim=128)

CASES = {
    # name: (config, cached rows before, prompt rows, what QKV, O, gate/up and down
    # take: F(ew rows) and K slices / row pairs per workgroup, or S(hort) tiles)
    "np1_rows11": (dict(ONE, ffn_dim=64), 0, 11, "F1/2 F1 F1/1 F1"),
    "np8_rows32": (dict(ONE, ffn_dim=2048), 0, 32, "F1/2 F1 F1/8 F4"),
    "np9_rows31": (dict(ONE, ffn_dim=2112), 5, 31, "F1/2 F1 F1/9 F4"),
    "np17_rows17": (dict(ONE, ffn_dim=4160), 0, 17, "F1/2 F1 F1/17 F8"),
    "np25_rows16": (dict(ONE, ffn_dim=6208), 3, 16, "F1/2 F1 F1/25 F8"),
    "np32_rows24": (dict(ONE, ffn_dim=8192), 0, 24, "F1/2 F1 F1/32 F8"),
    "np33_tiles": (dict(ONE, ffn_dim=8256), 0, 24, "F1/2 F1 S1 F8"),
    "rows33_tiles": (dict(ONE, ffn_dim=2048), 0, 33, "S1 S1 S1 S4"),
    "int8_np16": (dict(I8, ffn_dim=4096), 0, 32, "F1/2 F1 F1/16 F8"),
    "int8_np17": (dict(I8, ffn_dim=4160), 7, 23, "F1/2 F1 F1/17 F8"),
    "int8_np32": (dict(I8, ffn_dim=8192), 0, 12, "F1/2 F1 F1/32 F8"),
    # QKV np 24, ragged K stages (d 576), O split over K
    "qkv24": (dict(WIDE, d_model=576), 0, 23, "F1/24 F8 F1/4 F2"),
    "qkv24_int8": (dict(WIDE, d_model=576, wfmt="int8"), 2, 32, "F1/24 F8 F1/4 F2"),
    # QKV, O and down split over K; two layers
    "splits": (dict(d_model=2048, n_heads=16, n_kv_heads=8, head_dim=128, ffn_dim=4096), 0, 23, "F4/32 F4 F2/32 F8"),
    "splits_int8": (dict(d_model=2048, n_heads=32, n_kv_heads=8, ffn_dim=4096, wfmt="int8"), 0, 32, "F4/24 F4 F2/32 F8"),
    # odd head counts, d 320
    "ragged": (dict(d_model=320, ffn_dim=192, vocab=1000, n_heads=5, n_kv_heads=5), 0, 29, "F1/2 F1 F1/1 F1"),
    # a chunk of few rows behind a long one
    "behind_cache": (dict(ONE, ffn_dim=1024), 300, 20, "F1/2 F1 F1/4 F2"),
}


@pytest.mark.parametrize("name", list(CASES))
def test_prefill_few_rows(name, monkeypatch):
    kw, before, n, _ = CASES[name]
    kw = dict(kw, prompt_len=before + n, n_steps=8)
    monkeypatch.setitem(probe.CASES, name, (kw, before, n))
    probe.test_prefill_matches_sequential_oracle(name)
