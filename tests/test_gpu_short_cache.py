"""Decode, verify and short prefills behind a short cache give the bits on
record (needs an MI355X with 256 CUs).

Behind a few keys the new rows attend mostly to one another, so one cache entry
whose fp32 value rounds the other way moves everything after it: two equally
exact evaluations of a 7B verify of 4 rows at position 17 differ by 1e-3 in the
cache rows (each is as far from a 64-bit evaluation), at 2048 positions by 2e-4.
No bound below that holds there between two orders of the same sums, so up to
256 positions the kernels keep one order, and these digests (SHA-256 of logits,
tokens and written cache rows) pin it.  They are results of this library on one
compiler; an intended change of the order records them again:

    python -m tests.test_gpu_short_cache
"""
import hashlib
import json
import os

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "short_cache.json")

BASE = synth.CONFIGS["tiny"].with_(prompt_len=280, n_steps=16, prefill_by_model=False)

CONFIGS = {
    "tiny": dict(),
    "hd64_gqa2_int8": dict(n_heads=4, n_kv_heads=2, wfmt="int8"),
    "hd128_gqa4": dict(n_heads=4, n_kv_heads=1, head_dim=128),
    # three 256-k stages, the last one ragged
    "ragged_k": dict(d_model=576, ffn_dim=192),
    # eight query heads per kv head: the per-operation decode kernels
    "gqa8": dict(d_model=512, n_heads=8, n_kv_heads=1),
    # layers of the 1B and 7B shapes
    "1b_layers": dict(d_model=2048, n_heads=16, n_kv_heads=8, head_dim=128, ffn_dim=5632),
    "7b_layer": dict(n_layers=1, d_model=4096, n_heads=32, n_kv_heads=32, head_dim=128,
                     ffn_dim=11008),
    "7b_layer_int8": dict(n_layers=1, d_model=4096, n_heads=32, n_kv_heads=32, head_dim=128,
                          ffn_dim=11008, wfmt="int8"),
}

# (call, position, rows)
CALLS = [("verify", 17, 4), ("verify", 31, 2), ("verify", 100, 9), ("verify", 247, 9),
         ("verify", 246, 10), ("step", 0, 1), ("step", 17, 1), ("step", 128, 1), ("step", 255, 1),
         ("greedy", 60, 4), ("prefill", 0, 5), ("prefill", 200, 1)]


def digests(name):
    import torch

    from paper_2604_09752_amd.binding import DeviceModel

    cfg = BASE.with_(name="sc_" + name, **CONFIGS[name])
    kv = synth.make_kv(cfg)
    gpu = DeviceModel(cfg, synth.make_weights(cfg), kv_init=kv)
    toks = synth.make_prompt(cfg)
    logits = gpu.new_logits(cfg.max_verify)
    ids = torch.zeros(16, dtype=torch.int32, device=gpu.device)
    start = gpu.kv.clone()
    out = {}
    try:
        for call, pos, rows in CALLS:
            gpu.kv.copy_(start)
            torch.cuda.synchronize()
            t = [int(v) for v in toks[pos:pos + rows]]
            n = 1
            if call == "verify":
                gpu.verify(t[0], t[1:], pos, logits)
                n = rows
            elif call == "step":
                gpu.decode_step(t[0], pos, logits)
            elif call == "greedy":
                gpu.greedy(t[0], pos, rows, ids, logits)
            else:
                gpu.prefill(t, pos, logits)
            gpu.sync()
            h = hashlib.sha256(logits[:n].cpu().numpy().tobytes())
            h.update(np.ascontiguousarray(gpu.kv_rows(pos, pos + rows)).tobytes())
            if call == "greedy":
                h.update(ids[:rows].cpu().numpy().tobytes())
            out["%s %d rows at %d" % (call, rows, pos)] = h.hexdigest()[:16]
        assert gpu.status() == 0
    finally:
        gpu.close()
    return out


@pytest.mark.parametrize("name", list(CONFIGS))
def test_short_cache_bits(name):
    with open(GOLDEN) as f:
        want = json.load(f)[name]
    assert digests(name) == want


if __name__ == "__main__":
    rec = {n: digests(n) for n in CONFIGS}
    with open(GOLDEN, "w") as f:
        json.dump(rec, f, indent=1)
        f.write("\n")
