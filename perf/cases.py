"""Workloads by which the library's speed is followed, in the form its users run it.

Three kinds of case, all through the public entry points of paper_2505_00232_amd.binding:

"fc"      one quantized layer call (qfc_forward) on M token rows: the smallest unit of use.
"decode"  one token for each of up to 8 sequences through every operator of a decoder: embedding,
          per layer [normalization + QKV + rotary + cache append, attention, O + residual,
          normalization + gate+up with gated output, down + residual], then the LM head.
"tokens"  the same decoder for more than 8 token rows at once: S tokens of each of `batch`
          sequences that extend a context (prompts, chunks of prompts, and with S = 1 the decode step
          of more than 8 sequences, which ends with the LM head).

Weights are drawn with the bell shape that quantizing trained layers gives, scaled so that a layer keeps
the magnitude of its input and a quarter of it is added to the residual stream; caches and hidden states
are normal.  Shapes: the Llama-3.1-8B and
Gemma2-2B layers of this repository's benchmark, and generic ones.
"""
from __future__ import annotations

import math
import weakref

import torch

from paper_2505_00232_amd import binding as B

LLAMA = dict(hidden=4096, h_q=32, h_kv=8, d=128, ffn=14336, vocab=128256, gelu=False)
GEMMA = dict(hidden=2304, h_q=8, h_kv=4, d=256, ffn=9216, vocab=256000, gelu=True)

# Weight formats and prefill mode: (attention projections, feed-forward projections, LM head, int8 activations)
SCHEMES = {
    "g32": ("w4g32", "w4g32", "w8c", False),  # int4 in groups of 32, binary16 activations
    "w4c": ("w4c", "w4c", "w8c", False),      # int4 per channel, binary16 activations
    "q8": ("w8c", "w8c", "w8c", True),        # int8 per channel, int8 activations in prefill
    "844": ("w8c", "w4c", "w4c", True),       # int8 attention, int4 feed-forward and embedding
}
MODES = {"f16": B.QFC_COMPUTE_FP16_DEQUANT, "i8": B.QFC_COMPUTE_INT8_ACT, "i8_decode": B.QFC_COMPUTE_INT8_ACT_DECODE}


def listed():
    return [
        # a single small layer for one token: nothing but latency
        dict(name="fc_small", kind="fc", fmt="w8c", mode="i8", N=1024, K=512, M=1),
        # chat with one user: 1024 prompt tokens and up to 256 generated ones, whole model
        dict(name="decode_llama_g32", kind="decode", scheme="g32", layers=32, batch=1, context=1280, **LLAMA),
        # the paper's mixed 8/4/4 scheme on the smaller model (some of its layers), one user
        dict(name="decode_gemma_844", kind="decode", scheme="844", layers=8, batch=1, context=1280, **GEMMA),
        # one user with a long document in the cache
        dict(name="decode_llama_long", kind="decode", scheme="g32", layers=8, batch=1, context=12001, **LLAMA),
        # a small batch of users
        dict(name="decode_llama_844_b7", kind="decode", scheme="844", layers=8, batch=7, context=3000, **LLAMA),
        # servers with more users than the decode kernels' 8 rows
        dict(name="serve_llama_g32_b32", kind="tokens", scheme="g32", layers=4, batch=32, tokens=1, context=1500, **LLAMA),
        dict(name="serve_llama_q8_b20", kind="tokens", scheme="q8", layers=2, batch=20, tokens=1, context=1500, **LLAMA),
        # a short question
        dict(name="prompt_gemma_g32_77", kind="tokens", scheme="g32", layers=4, batch=1, tokens=77, context=77, **GEMMA),
        # a chunk of a long prompt behind the chunks before it
        dict(name="chunk_llama_844_300", kind="tokens", scheme="844", layers=2, batch=1, tokens=300, context=6300, **LLAMA),
        # the prompt of the paper's measurements
        dict(name="prefill_llama_q8_1024", kind="tokens", scheme="q8", layers=2, batch=1, tokens=1024, context=1024, **LLAMA),
        dict(name="prefill_gemma_g32_2048", kind="tokens", scheme="g32", layers=2, batch=1, tokens=2048, context=2048, **GEMMA),
        # a long document read at once
        dict(name="prefill_llama_w4c_6000", kind="tokens", scheme="w4c", layers=1, batch=1, tokens=6000, context=6000, **LLAMA),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _family(rng):
    pick = rng.random()
    if pick < 0.3:
        return dict(LLAMA)
    if pick < 0.6:
        return dict(GEMMA)
    d = rng.choice([64, 128, 256])
    h_kv = rng.choice([1, 2, 4, 8])
    g = rng.choice([1, 2, 4, 8]) if h_kv * d <= 512 else rng.choice([1, 2, 4])
    return dict(hidden=128 * rng.randint(6, 32), h_q=h_kv * g, h_kv=h_kv, d=d, ffn=32 * rng.randint(64, 448),
                vocab=_log_int(rng, 8000, 131072), gelu=rng.random() < 0.5)


def draw(rng):
    pick = rng.random()
    if pick < 0.3:
        fmt = rng.choice(["w8c", "w4g32", "w4c"])
        mode = "f16" if fmt == "w4g32" else rng.choice(["f16", "i8", "i8", "i8_decode"])
        M = rng.randint(1, 8) if mode == "i8_decode" else _log_int(rng, 1, 4096)
        return dict(kind="fc", fmt=fmt, mode=mode, N=_log_int(rng, 200, 32768), K=32 * _log_int(rng, 8, 448), M=M)
    scheme = rng.choice(sorted(SCHEMES))
    if pick < 0.6:
        return dict(kind="decode", scheme=scheme, layers=rng.randint(2, 6), batch=rng.randint(1, 8),
                    context=_log_int(rng, 64, 16384), **_family(rng))
    if pick < 0.75:
        return dict(kind="tokens", scheme=scheme, layers=rng.randint(1, 2), batch=_log_int(rng, 9, 96), tokens=1,
                    context=_log_int(rng, 64, 3000), **_family(rng))
    tokens = _log_int(rng, 17, 4096)
    past = 0 if rng.random() < 0.6 else _log_int(rng, 64, 6000)
    return dict(kind="tokens", scheme=scheme, layers=1 if tokens > 1500 else 2, batch=1, tokens=tokens,
                context=past + tokens, **_family(rng))


def _generator(seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return gen


def _linear(gen, N, K, fmt, mode, pairs=False, gain=1.0):
    sigma = 28.0 if fmt == "w8c" else 2.5
    lo, hi = (-127, 127) if fmt == "w8c" else (-8, 7)
    codes = torch.randn((N, K), generator=gen, device="cuda").mul_(sigma).round_().clamp_(lo, hi).to(torch.int8)
    shape = (N, K // 32) if fmt == "w4g32" else (N,)
    scales = torch.rand(shape, generator=gen, device="cuda").mul_(0.4).add_(0.8).mul_(gain / (sigma * math.sqrt(K)))
    return B.QuantLinear(codes, scales.half() if fmt == "w4g32" else scales, fmt, mode, max_m=1, gated_pairs=pairs)


def _close_with(owner, linears):
    for l in linears:
        weakref.finalize(owner, l.close).atexit = False


def _normal(gen, *shape):
    return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float16)


class _Decoder:
    """What an inference program keeps: packed layers, caches, tables and buffers."""

    def __init__(self, case, seed):
        gen = _generator(seed)
        c = self.case = dict(case)
        attn_fmt, ffn_fmt, head_fmt, i8 = SCHEMES[c["scheme"]]
        mode = B.QFC_COMPUTE_INT8_ACT if i8 else B.QFC_COMPUTE_FP16_DEQUANT
        self.i8 = i8
        hidden, h_q, h_kv, d, ffn = c["hidden"], c["h_q"], c["h_kv"], c["d"], c["ffn"]
        batch, S = c["batch"], c.get("tokens", 1)
        M = self.M = batch * S
        self.S = S
        self.offset = 1.0 if c["gelu"] else 0.0
        self.act_fn = B.QFC_ACT_GELU_TANH if c["gelu"] else B.QFC_ACT_SILU
        C = (c["context"] + 63) // 64 * 64
        self.pos0 = c["context"] - S
        self.shape = B.AttnShape(batch, h_q, h_kv, d, C)
        G = batch * h_kv
        self.layers = []
        for _ in range(c["layers"]):
            self.layers.append((
                _linear(gen, (h_q + 2 * h_kv) * d, hidden, attn_fmt, mode),
                _linear(gen, hidden, h_q * d, attn_fmt, mode, gain=0.25),
                _linear(gen, 2 * ffn, hidden, ffn_fmt, mode, pairs=True),
                _linear(gen, hidden, ffn, ffn_fmt, mode, gain=0.25)))
        self.with_head = S == 1
        # the LM head is the embedding table too: rows large enough for a residual stream
        self.head = _linear(gen, c["vocab"], hidden, head_fmt, B.QFC_COMPUTE_INT8_ACT, gain=16.0) if self.with_head else None
        # one workspace for all layers, whose calls follow each other on one stream
        linears = [l for layer in self.layers for l in layer] + ([self.head] if self.head else [])
        self.workspace = torch.empty(max(B.qfc_workspace_size(l.handle, M) for l in linears), dtype=torch.uint8, device="cuda")
        for l in linears:
            l.workspace = self.workspace
            B.qfc_bind_workspace(l.handle, self.workspace)
        _close_with(self, linears)
        norm = lambda: (1.0 - self.offset + 0.1 * _normal(gen, hidden)).half()
        self.gammas = [(norm(), norm()) for _ in range(c["layers"])]
        self.final_gamma = norm()
        self.kcache = _normal(gen, c["layers"], G, C, d)
        self.vcache = _normal(gen, c["layers"], G, C // 64, d, 64)
        self.table = B.qfc_rope_table(self.shape, 500000.0, C)
        self.ids = torch.randint(0, c["vocab"], (M,), generator=gen, device="cuda", dtype=torch.int32)
        self.x = _normal(gen, M, hidden)
        E = lambda *s: torch.empty(s, dtype=torch.float16, device="cuda")
        self.qkv, self.normed = E(batch, S, (h_q + 2 * h_kv) * d), E(M, hidden)
        self.q, self.att = E(G, S * (h_q // h_kv), d), E(G, S * (h_q // h_kv), d)
        self.h1, self.h2, self.act = E(M, hidden), (E(M, hidden), E(M, hidden)), E(M, ffn)
        self.logits = E(M, c["vocab"]) if self.with_head else None
        self.attn_ws = torch.empty(B.qfc_attention_workspace_size(self.shape, S), dtype=torch.uint8, device="cuda")

    def decode(self):
        c, M, n_ctx = self.case, self.M, self.case["context"]
        h = self.x
        B.qfc_embedding(self.head.handle, self.ids, h)
        for i, (qkv, o, gate_up, down) in enumerate(self.layers):
            g1, g2 = self.gammas[i]
            B.qfc_forward_qkv_rope(qkv.handle, h, self.pos0, self.shape, self.table, self.q, self.kcache[i], self.vcache[i],
                                   norm_gamma=g1, norm_eps=1e-5, norm_offset=self.offset)
            B.qfc_attention(self.q, self.kcache[i], self.vcache[i], 1, n_ctx, self.shape, self.attn_ws, self.att)
            B.qfc_forward_fused(o.handle, self.att.view(M, c["h_q"] * c["d"]), self.h1, residual=h)
            B.qfc_forward_fused(gate_up.handle, self.h1, self.act, activation=self.act_fn, gated_output=True,
                                norm_gamma=g2, norm_eps=1e-5, norm_offset=self.offset)
            h = self.h2[i % 2]
            B.qfc_forward_fused(down.handle, self.act, h, residual=self.h1)
        B.qfc_forward_fused(self.head.handle, h, self.logits, norm_gamma=self.final_gamma, norm_eps=1e-5, norm_offset=self.offset)
        return {"logits": self.logits, "kcache": self.kcache, "vcache": self.vcache}

    def _normed_forward(self, layer, h, gamma, out):
        if self.i8:  # the normalization leaves the quantized activations where the layer reads them
            B.qfc_rmsnorm(h, gamma, 1e-5, self.offset, consumer=layer.handle)
            B.qfc_forward_q8(layer.handle, None, None, out)
        else:
            B.qfc_rmsnorm(h, gamma, 1e-5, self.offset, y=self.normed)
            B.qfc_forward(layer.handle, self.normed, out)

    def tokens(self):
        c, M, S, n_ctx = self.case, self.M, self.S, self.case["context"]
        batch, h_q, h_kv, d = c["batch"], c["h_q"], c["h_kv"], c["d"]
        h = self.x
        if self.with_head:
            B.qfc_embedding(self.head.handle, self.ids, h)
        for i, (qkv, o, gate_up, down) in enumerate(self.layers):
            g1, g2 = self.gammas[i]
            self._normed_forward(qkv, h, g1, self.qkv.view(M, -1))
            B.qfc_rope_qkv(self.qkv, self.pos0, self.shape, 500000.0, self.q, self.kcache[i], self.vcache[i])
            B.qfc_attention(self.q, self.kcache[i], self.vcache[i], S, n_ctx, self.shape, self.attn_ws, self.att)
            rows = self.att if S == 1 else self.att.view(batch, h_kv, S, h_q // h_kv, d).transpose(1, 2).contiguous()
            B.qfc_forward_fused(o.handle, rows.view(M, h_q * d), self.h1, residual=h)
            B.qfc_rmsnorm(self.h1, g2, 1e-5, self.offset, y=self.normed)
            B.qfc_forward_fused(gate_up.handle, self.normed, self.act, activation=self.act_fn, gated_output=True)
            h = self.h2[i % 2]
            B.qfc_forward_fused(down.handle, self.act, h, residual=self.h1)
        if self.with_head:
            B.qfc_rmsnorm(h, self.final_gamma, 1e-5, self.offset, consumer=self.head.handle)
            B.qfc_forward_q8(self.head.handle, None, None, self.logits)
            h = self.logits
        return {"out": h, "kcache": self.kcache, "vcache": self.vcache}


class _Layer:
    def __init__(self, case, seed):
        gen = _generator(seed)
        self.layer = _linear(gen, case["N"], case["K"], case["fmt"], MODES[case["mode"]])
        self.workspace = torch.empty(B.qfc_workspace_size(self.layer.handle, case["M"]), dtype=torch.uint8, device="cuda")
        B.qfc_bind_workspace(self.layer.handle, self.workspace)
        _close_with(self, [self.layer])
        self.x = _normal(gen, case["M"], case["K"])
        self.y = torch.empty((case["M"], case["N"]), dtype=torch.float16, device="cuda")

    def forward(self):
        B.qfc_forward(self.layer.handle, self.x, self.y)
        return self.y


def prepare(case, seed):
    return _Layer(case, seed) if case["kind"] == "fc" else _Decoder(case, seed)


def run(state):
    if isinstance(state, _Layer):
        return state.forward()
    return state.decode() if state.case["kind"] == "decode" else state.tokens()


def _fc_work(fmt, N, K, M):
    weights = {"w8c": N * K + 4 * N, "w4c": N * K // 2 + 4 * N, "w4g32": N * K // 2 + N * K // 16}[fmt]
    return weights + 2 * M * (N + K), 2 * M * N * K


def work(case):
    if case["kind"] == "fc":
        b, f = _fc_work(case["fmt"], case["N"], case["K"], case["M"])
        return {"bytes": b, "flops": f}
    c, S = case, case.get("tokens", 1)
    M = c["batch"] * S
    attn_fmt, ffn_fmt, head_fmt, _ = SCHEMES[c["scheme"]]
    h_q, h_kv, d, hidden, ffn, n = c["h_q"], c["h_kv"], c["d"], c["hidden"], c["ffn"], c["context"]
    parts = [_fc_work(attn_fmt, (h_q + 2 * h_kv) * d, hidden, M), _fc_work(attn_fmt, hidden, h_q * d, M),
             _fc_work(ffn_fmt, 2 * ffn, hidden, M), _fc_work(ffn_fmt, hidden, ffn, M)]
    # cache read once; token s of a sequence sees n - S + 1 + s positions
    seen = S * (n - S) + S * (S + 1) // 2
    parts.append((4 * c["batch"] * h_kv * n * d + 4 * M * h_q * d, 4 * c["batch"] * h_q * d * seen))
    nbytes, flops = (c["layers"] * sum(p[i] for p in parts) for i in (0, 1))
    nbytes -= c["layers"] * 2 * M * ffn  # the gated output is half as wide as the layer
    if S == 1:
        b, f = _fc_work(head_fmt, c["vocab"], hidden, M)
        nbytes, flops = nbytes + b, flops + f
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times the 2-norm difference from a 64-bit evaluation (same quantized weights and
    activations).  One layer: 2.1e-4 to 2.9e-4.  A decoder's binary16 roundings add up over its layers
    (decode: 1.2e-3 for 8 layers, 3.6e-3 for 32; prompts: 1.6e-4 to 5.6e-4).  Where activations are
    quantized, a rounding that flips moves an 8-bit code and the layers behind it see that step:
    4.0e-3 to 5.0e-3 for prompts of two layers, 4.6e-3 (one quantization, before the LM head) to
    2.1e-2 with the LM head behind two quantized layers."""
    if case["kind"] == "fc":
        return {"rel": 1.2e-3}
    i8 = SCHEMES[case["scheme"]][3]
    if case["kind"] == "decode":
        return {"rel": 1.5e-2}
    if case["tokens"] == 1:
        return {"rel": 8e-2 if i8 else 2e-2}
    return {"rel": 2e-2 if i8 else 2.5e-3}
