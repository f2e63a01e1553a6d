"""A handle's results do not depend on what its workspace held before the load
(needs an MI355X): the arrival counters of verify, prefill and attention are
cleared for every handle, also for shapes and settings without the step kernel."""
import numpy as np
import pytest
import torch

import synth
from tests.gpu_cases import env_set

pytestmark = pytest.mark.gpu

BASE = synth.CONFIGS["tiny"].with_(n_layers=2, prompt_len=96, n_steps=16)

CASES = {
    # O and down of prefill and verify split over K
    "step_kernel": (dict(d_model=1024, ffn_dim=4096, n_heads=8, n_kv_heads=8, head_dim=128), "1"),
    "per_op": (dict(d_model=1024, ffn_dim=4096, n_heads=8, n_kv_heads=8, head_dim=128), "0"),
    # eight query heads per kv head: never the step kernel
    "gqa8": (dict(d_model=512, n_heads=8, n_kv_heads=1), "1"),
}


def _results(gpu, toks):
    logits = gpu.new_logits(10)
    out = []
    # prompts of few rows and in tiles, verify, a step
    for rows, pos in ((70, 0), (23, 70), (9, 60)):
        if rows == 9:
            gpu.verify(toks[pos], toks[pos + 1:pos + rows], pos, logits)
        else:
            gpu.prefill(toks[pos:pos + rows], pos, logits)
        gpu.sync()
        out.append(logits[:rows if rows == 9 else 1].cpu().numpy().copy())
        out.append(gpu.kv_rows(pos, pos + rows))
    gpu.decode_step(toks[0], 93, logits)
    gpu.sync()
    out.append(logits[0].cpu().numpy().copy())
    return out


@pytest.mark.parametrize("fill", [0xFF, 0x01])
@pytest.mark.parametrize("name", list(CASES))
def test_workspace_contents_do_not_matter(name, fill):
    from paper_2604_09752_amd import binding as B

    kw, mega = CASES[name]
    cfg = BASE.with_(name="ws_" + name, **kw)
    toks = [int(t) for t in synth.make_prompt(cfg)]
    with env_set(AIO_MEGA=mega):
        gpu = B.DeviceModel(cfg, synth.make_weights(cfg))
        try:
            want = _results(gpu, toks)
            B.aio_model_free(gpu.handle)
            gpu.handle = None
            gpu.kv.zero_()
            gpu.ws.fill_(fill)
            torch.cuda.synchronize()
            gpu.handle = B.aio_model_load(gpu.c, gpu._w, gpu.kv, gpu.ws, gpu.stream.cuda_stream)
            got = _results(gpu, toks)
            assert gpu.status() == 0
        finally:
            gpu.close()
    for w, g in zip(want, got):
        assert np.array_equal(w.view(np.uint8), g.view(np.uint8))
