"""A prefill's residual product rounds x once, however its K is split (needs an
MI355X): the slices' sums are added to one another first.

x is 1 everywhere.  The O projection adds eight K slices of 0.3 ulp each to the
even columns: 2.4 ulp in all, where slice by slice every sum would round back to
1.  The LM head's first row is column 0 minus column 1, so its logit is what the
product added; it may be off by the one rounding of x (half an ulp) and by the
fp32 errors of the sums (1e-5 of them)."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

ULP = 2.0 ** -23  # of x = 1


def _bf16(v):
    return np.uint16(np.float32(v).view(np.uint32) >> 16)


@pytest.mark.parametrize("rows", [11, 32, 33])
def test_residual_is_rounded_once(rows):
    from paper_2604_09752_amd.binding import DeviceModel

    # K of O is 4096: eight slices of 512 for up to 32 rows
    cfg = synth.CONFIGS["tiny"].with_(name="residual", n_layers=1, d_model=256, n_heads=32,
                                      n_kv_heads=4, head_dim=128, ffn_dim=64, vocab=64,
                                      prompt_len=64, n_steps=8)
    d, one = cfg.d_model, _bf16(1.0)
    w = {"embed": np.full((cfg.vocab, d), one, np.uint16),
         "final_norm": np.full(d, one, np.uint16),
         "lm_head": np.zeros((cfg.vocab, d), np.uint16),
         "layers.0.attn_norm": np.full(d, one, np.uint16),
         "layers.0.ffn_norm": np.full(d, one, np.uint16)}
    for n, shape in synth.linear_shapes(cfg).items():
        w["layers.0." + n] = np.zeros(shape, np.uint16)
    w["lm_head"][0, 0], w["lm_head"][0, 1] = one, _bf16(-1.0)
    # every value entry is v (wv v / d, a power of two apart), and so is o
    v_bits = _bf16(0.3 * 2.0 ** -12)
    v = float(synth.bf16_bits_to_f32(np.array([v_bits]))[0])
    w["layers.0.wv"][:] = _bf16(v / d)
    w["layers.0.wo"][0::2, :] = _bf16(2.0 ** -20)
    added = 4096 * 2.0 ** -20 * v
    assert 2.3 * ULP < added < 2.45 * ULP

    gpu = DeviceModel(cfg, w)
    try:
        logits = gpu.new_logits(1)
        gpu.prefill([1] * rows, 0, logits)
        gpu.sync()
        got = float(logits[0, 0])
        assert gpu.status() == 0
    finally:
        gpu.close()
    assert abs(got - added) <= 0.5 * ULP + 1e-5 * added, (got / ULP, added / ULP)
