"""Timed cases of the batch-1 decoder: what a program that serves one request
at a time has the library do.

Three kinds of call, each through the C ABI's Python binding:

* ``step`` / ``greedy``: decode, one token with its logits
  (``aio_decode_step``) or a device-resident run of tokens
  (``aio_decode_greedy``);
* ``verify``: one forward of the current token plus k prompt-lookup drafts and
  the argmax of every row (``aio_verify``, ``aio_argmax``);
* ``prefill``: a prompt into the cache and its last token's logits
  (``aio_prefill``); for the probe also the entropy of the category labels
  (``aio_category_entropy``).

The models are the repository's own workloads: the tiny decoder of its tests,
the 1B-class probe and the 7B-class backbone, with bf16 or W8A16 weights
(int8 rows quantised by their largest magnitude, fp16 scales).  Weights are
N(0, 0.02), gains close to one, cached keys and values N(0, 1).

Every pass returns its logits whole, what it derived from them, and the rows
of the KV cache that it wrote (all layers, heads and positions written).
"""
from __future__ import annotations

import ctypes
import math

import numpy as np
import torch

from paper_2604_09752_amd import binding as aio

SHAPES = {
    "tiny": dict(n_layers=2, d_model=256, n_heads=4, n_kv_heads=4, head_dim=64, ffn_dim=1024,
                 vocab=4096),
    "1b": dict(n_layers=24, d_model=2048, n_heads=16, n_kv_heads=8, head_dim=128, ffn_dim=5632,
               vocab=32000),
    "7b": dict(n_layers=32, d_model=4096, n_heads=32, n_kv_heads=32, head_dim=128, ffn_dim=11008,
               vocab=32000),
}
LABELS = 4  # category label tokens of the probe
RMS_EPS = 1e-5
ROPE_BASE = 10000.0
LINEARS = ("wq", "wk", "wv", "wo", "w_gate", "w_up", "w_down")


def _case(model, kind, pos, rows, wfmt="bf16", name=None):
    c = {"model": model, "kind": kind, "wfmt": wfmt, "pos": pos, "rows": rows}
    c.update(SHAPES[model])
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: one token of a toy decoder, all latency
        _case("tiny", "step", 128, 1, name="step_tiny_128"),
        # the probe / small model generating after a 2K prompt
        _case("1b", "greedy", 2048, 8, name="greedy_1b_2k"),
        # the backbone generating after a 2K prompt, bf16 and W8A16 weights
        _case("7b", "greedy", 2048, 4, name="greedy_7b_2k"),
        _case("7b", "greedy", 2048, 4, wfmt="int8", name="greedy_7b_int8_2k"),
        # one token at the long context the backbone is kept for
        _case("7b", "step", 32768, 1, name="step_7b_32k"),
        # prompt lookup with a look-ahead of 2 on the small model
        _case("1b", "verify", 1531, 3, name="verify_1b_k2"),
        # prompt lookup with 8 drafts on the backbone, bf16 and W8A16 weights
        _case("7b", "verify", 2048, 9, name="verify_7b_2k_k8"),
        _case("7b", "verify", 2048, 9, wfmt="int8", name="verify_7b_int8_2k_k8"),
        # the probe's forward over a short templated request
        _case("1b", "prefill", 0, 23, name="prefill_1b_23"),
        # ... over an ordinary request of a ragged length
        _case("1b", "prefill", 0, 389, name="prefill_1b_389"),
        # ... over the longest request the small model is routed
        _case("1b", "prefill", 0, 2048, name="prefill_1b_2048"),
        # the backbone's prompt
        _case("7b", "prefill", 0, 1000, name="prefill_7b_1000"),
    ]


def _log_int(rng, lo, hi):
    return min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))


def draw(rng):
    kind = rng.choice(["step", "greedy", "verify", "prefill"])
    model = rng.choice(["tiny", "1b", "7b"])
    wfmt = rng.choice(["bf16", "int8"])
    ctx = 2048 if model == "tiny" else 32768
    if kind == "prefill":
        # the longer prompts on the small models, whose cost stays below the
        # backbone's listed prompt; some continue an earlier turn's cache
        rows = _log_int(rng, 11, 700 if model == "7b" else 2048)
        pos = _log_int(rng, 1, 1024) if rng.random() < 0.3 else 0
    elif kind == "verify":
        rows, pos = rng.randint(2, 10), _log_int(rng, 16, ctx // 2)
    elif kind == "greedy":
        rows, pos = rng.randint(2, 6), _log_int(rng, 16, ctx // 4)
    else:
        rows, pos = 1, _log_int(rng, 16, ctx)
    return _case(model, kind, pos, rows, wfmt)


# ------------------------------------------------------------------ inputs

def _max_ctx(case):
    return case["pos"] + case["rows"] + 64


def _weights(case, gen, device):
    """Name -> device tensor, every linear [out][in]."""
    d, F, V, hd = case["d_model"], case["ffn_dim"], case["vocab"], case["head_dim"]
    q, kv = case["n_heads"] * hd, case["n_kv_heads"] * hd

    def normal(*shape, mean=0.0, std=0.02):
        return torch.empty(shape, dtype=torch.bfloat16, device=device).normal_(mean, std,
                                                                               generator=gen)

    out = {}

    def linear(name, n, k):
        w = normal(n, k)
        if case["wfmt"] == "int8":
            w = w.float()
            s = (w.abs().amax(dim=1) / 127.0).half()
            out[name + ".scale"] = s
            w = (w / s.float()[:, None]).round_().clamp_(-127, 127).to(torch.int8)
        out[name] = w

    out["embed"] = normal(V, d)
    for l in range(case["n_layers"]):
        p = "layers.%d." % l
        out[p + "attn_norm"] = normal(d, mean=1.0)
        out[p + "ffn_norm"] = normal(d, mean=1.0)
        for n, shape in zip(LINEARS, ((q, d), (kv, d), (kv, d), (d, q), (F, d), (F, d), (d, F))):
            linear(p + n, *shape)
    out["final_norm"] = normal(d, mean=1.0)
    linear("lm_head", V, d)
    return out


def _inputs(case, seed, device):
    gen = torch.Generator(device=device)
    gen.manual_seed(seed)
    w = _weights(case, gen, device)
    kv = torch.zeros((case["n_layers"], 2, case["n_kv_heads"], _max_ctx(case), case["head_dim"]),
                     dtype=torch.bfloat16, device=device)
    kv[..., : case["pos"], :].normal_(0.0, 1.0, generator=gen)
    rs = np.random.RandomState(seed % (2 ** 32))
    n = 1 if case["kind"] in ("step", "greedy") else case["rows"]
    tokens = rs.randint(0, case["vocab"], size=n).astype(np.int32)
    labels = rs.choice(case["vocab"], size=LABELS, replace=False).astype(np.int32)
    return w, kv, tokens, labels


class _State:
    """A loaded model, its buffers and the request's tokens."""

    def __init__(self, case, seed):
        self.device = torch.device("cuda", torch.cuda.current_device())
        self.case = case
        self.w, self.kv, self.tokens, self.labels = _inputs(case, seed, self.device)
        c = aio.aio_config()
        for n in ("n_layers", "d_model", "n_heads", "n_kv_heads", "head_dim", "ffn_dim", "vocab"):
            setattr(c, n, case[n])
        c.max_ctx, c.max_verify = _max_ctx(case), aio.AIO_MAX_VERIFY_ROWS
        int8 = case["wfmt"] == "int8"
        c.wfmt = aio.AIO_WFMT_INT8 if int8 else aio.AIO_WFMT_BF16
        c.rms_eps, c.rope_base = RMS_EPS, ROPE_BASE
        assert self.kv.numel() * 2 == aio.aio_kv_bytes(c)
        self.ws = torch.zeros(aio.aio_workspace_bytes(c), dtype=torch.uint8, device=self.device)
        layers = (aio.aio_layer_weights * c.n_layers)()
        for l in range(c.n_layers):
            p = "layers.%d." % l
            layers[l].attn_norm = self.w[p + "attn_norm"].data_ptr()
            layers[l].ffn_norm = self.w[p + "ffn_norm"].data_ptr()
            for n, s in zip(aio.LINEARS, aio.SCALES):
                setattr(layers[l], n, self.w[p + n].data_ptr())
                if int8:
                    setattr(layers[l], s, self.w[p + n + ".scale"].data_ptr())
        w = aio.aio_weights()
        w.embed = self.w["embed"].data_ptr()
        w.final_norm = self.w["final_norm"].data_ptr()
        w.lm_head = self.w["lm_head"].data_ptr()
        if int8:
            w.s_lm_head = self.w["lm_head.scale"].data_ptr()
        w.layers = ctypes.cast(layers, ctypes.POINTER(aio.aio_layer_weights))
        self.handle = aio.aio_model_load(c, w, self.kv, self.ws,
                                         torch.cuda.current_stream().cuda_stream)
        rows = case["rows"] if case["kind"] == "verify" else 1
        self.logits = torch.empty((rows, case["vocab"]), dtype=torch.float32, device=self.device)
        self.ids = torch.zeros(case["rows"], dtype=torch.int32, device=self.device)
        self.entropy = torch.zeros(2, dtype=torch.float32, device=self.device)

    def __del__(self):
        if getattr(self, "handle", None):
            aio.aio_model_free(self.handle)
            self.handle = None


def prepare(case, seed):
    return _State(case, seed)


def run(state):
    case, h, pos, rows = state.case, state.handle, state.case["pos"], state.case["rows"]
    out = {"logits": state.logits, "kv_rows": state.kv[..., pos: pos + rows, :]}
    if case["kind"] == "step":
        aio.aio_decode_step(h, int(state.tokens[0]), pos, state.logits)
    elif case["kind"] == "greedy":
        aio.aio_decode_greedy(h, int(state.tokens[0]), pos, rows, state.ids, state.logits)
        out["ids"] = state.ids
    elif case["kind"] == "verify":
        aio.aio_verify(h, int(state.tokens[0]), state.tokens[1:], rows - 1, pos, state.logits)
        aio.aio_argmax(h, state.logits, rows, case["vocab"], state.ids)
        out["ids"] = state.ids
    else:
        rc = aio.lib().aio_prefill(h, state.tokens.ctypes.data, rows, pos,
                                   state.logits.data_ptr())
        if rc != aio.AIO_OK:
            raise aio.AioError(rc, "aio_prefill")
        aio.aio_category_entropy(h, state.logits, state.labels, state.entropy)
        out["entropy"] = state.entropy
    return out


# ------------------------------------------------------------ bytes and flops

def work(case):
    d, F, V, L = case["d_model"], case["ffn_dim"], case["vocab"], case["n_layers"]
    q, kv = case["n_heads"] * case["head_dim"], case["n_kv_heads"] * case["head_dim"]
    pos, rows = case["pos"], case["rows"]
    layer = d * (q + 2 * kv) + q * d + 3 * d * F
    outs = L * (q + 2 * kv + 2 * F + 2 * d) + V
    int8 = case["wfmt"] == "int8"
    wbytes = (L * layer + V * d) * (1 if int8 else 2) + (2 * outs if int8 else 0)
    wbytes += 2 * (2 * L + 1) * d
    row = 2 * L * kv * 2                      # K and V of one position, all layers
    heads = rows if case["kind"] == "verify" else 1
    # a score and a weighted value per query, visible key and dimension
    seen = rows * pos + rows * (rows + 1) // 2
    flops = 2 * rows * L * layer + 4 * L * q * seen
    if case["kind"] == "greedy":              # every token reads the weights and the cache
        nbytes = rows * (wbytes + 2 * d + row) + row * seen + 4 * V
        flops += 2 * rows * V * d
    else:
        nbytes = wbytes + rows * (2 * d + row) + row * pos + 4 * V * heads
        flops += 2 * heads * V * d
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # The cache rows set the bound: they are bf16, and a value near a rounding
    # boundary may land on either side of it (at most 2^-7 of itself).  Behind
    # a cache that is given, the share that does puts a pass's rows within
    # 2e-4 of the 64-bit evaluation's and its logits within 2e-5.  A prompt's
    # rows attend to one another's rounded rows, layer after layer: 2e-3 and
    # 1.3e-3.
    if case["kind"] == "prefill":
        return {"rel": 8e-3, "max": 5e-2}
    return {"rel": 6e-4, "max": 2e-2}


# --------------------------------------------------------- 64-bit evaluation

def exact(case, seed):
    device = torch.device("cuda", torch.cuda.current_device())
    w, cache, tokens, labels = _inputs(case, seed, device)
    d, V, hd = case["d_model"], case["vocab"], case["head_dim"]
    H, Hkv, L = case["n_heads"], case["n_kv_heads"], case["n_layers"]
    half, f64 = hd // 2, torch.float64
    inv = ROPE_BASE ** (-2.0 * torch.arange(half, dtype=f64, device=device) / hd)

    def mul(name, x):
        y = x @ w[name].to(f64).t()
        return y * w[name + ".scale"].to(f64) if name + ".scale" in w else y

    def norm(x, g):
        return x * torch.rsqrt((x * x).mean(dim=-1, keepdim=True) + RMS_EPS) * w[g].to(f64)

    def forward(toks, pos):
        """The rows' final residual; their K and V go to the cache (bf16)."""
        n = len(toks)
        x = w["embed"][torch.as_tensor(toks, device=device).long()].to(f64)
        p = torch.arange(pos, pos + n, dtype=f64, device=device)
        phi = p[:, None] * inv
        # the rotation's table is 32-bit
        cos, sin = phi.cos().float().to(f64), phi.sin().float().to(f64)

        def rope(t):  # [heads][n][hd]
            a, b = t[..., :half], t[..., half:]
            return torch.cat((a * cos - b * sin, b * cos + a * sin), dim=-1)

        hidden = (torch.arange(pos + n, device=device)[None, :] >
                  torch.arange(pos, pos + n, device=device)[:, None])
        for l in range(L):
            pre = "layers.%d." % l
            h = norm(x, pre + "attn_norm")
            heads = [mul(pre + m, h).view(n, -1, hd).transpose(0, 1).contiguous()
                     for m in ("wq", "wk", "wv")]
            q = rope(heads[0])
            cache[l, 0, :, pos: pos + n] = rope(heads[1]).to(torch.bfloat16)
            cache[l, 1, :, pos: pos + n] = heads[2].to(torch.bfloat16)
            att = torch.empty((n, H, hd), dtype=f64, device=device)
            for g in range(Hkv):
                k = cache[l, 0, g, : pos + n].to(f64)
                v = cache[l, 1, g, : pos + n].to(f64)
                for j in range(g * (H // Hkv), (g + 1) * (H // Hkv)):
                    s = (q[j] @ k.t()) / math.sqrt(hd)
                    s.masked_fill_(hidden, -math.inf)
                    att[:, j] = torch.softmax(s, dim=-1) @ v
            x = x + mul(pre + "wo", att.view(n, H * hd))
            h = norm(x, pre + "ffn_norm")
            g = mul(pre + "w_gate", h)
            x = x + mul(pre + "w_down", g * torch.sigmoid(g) * mul(pre + "w_up", h))
        return x

    def head(x):
        return mul("lm_head", norm(x, "final_norm"))

    pos, rows = case["pos"], case["rows"]
    out = {}
    if case["kind"] == "greedy":
        ids = []
        tok = int(tokens[0])
        for s in range(rows):
            logits = head(forward([tok], pos + s))
            tok = int(logits[0].argmax())
            ids.append(tok)
        out["logits"] = logits
        out["ids"] = torch.tensor(ids, dtype=torch.int32, device=device)
    else:
        x = forward(tokens, pos)
        out["logits"] = head(x if case["kind"] == "verify" else x[-1:])
        if case["kind"] == "verify":
            out["ids"] = out["logits"].argmax(dim=-1).to(torch.int32)
        elif case["kind"] == "prefill":
            t = out["logits"][0, torch.as_tensor(labels, device=device).long()]
            p = torch.softmax(t, dim=0)
            out["entropy"] = torch.stack((-(p * p.log()).sum(), t.argmax().to(f64)))
    out["kv_rows"] = cache[..., pos: pos + rows, :].to(f64)
    return out
