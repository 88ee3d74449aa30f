"""What programs have this library do, as cases that can be timed: whole encoder forwards from one short sentence to the
largest serving batch, single layers, an FFN block over packed tokens, and the non-linear kernels on their own.

Shapes are the repository's configurations (`synth.CONFIGS`, the latency grid and the stand-alone kernel shapes of
`bench.py`) and, between them, the sizes that text gives: batches padded to their longest sentence, which is hardly ever a
multiple of anything, and token counts that are sums of sentence lengths.  Weights, scales and activations follow the
distributions of `synth`; everything is made from the case and the seed.  All outputs are INT8 / INT16 and exact.
"""
import math

import numpy as np
import torch

from paper_2101_01321_amd import binding as B
from paper_2101_01321_amd import synth

# model -> hidden, heads, ffn, layers
MODELS = {"tiny": (256, 4, 1024, 1), "base": (768, 12, 3072, 12), "large": (1024, 16, 4096, 24)}
VOCAB, MAX_SEQ, MAX_TOKENS = 50265, 512, 32768
S_ACT = synth.LN_OUT_ALPHA / 127.0           # scale of a LayerNorm output: what every layer and FFN block is fed


def listed():
    return [
        # the smallest unit a program calls: one small layer on one sequence; almost all launch latency
        {"name": "layer_tiny", "kind": "layer", "model": "tiny", "batch": 1, "seq": 128},
        # one Base layer on a few short sentences through the entry point that needs no workspace
        {"name": "layer_base_static_b3", "kind": "layer", "model": "base", "batch": 3, "seq": 59},
        # interactive serving: one sequence, the forward captured once in a HIP graph and replayed
        {"name": "base_b1_graph", "kind": "encoder", "model": "base", "batch": 1, "seq": 128, "input": "activations", "graph": True},
        # a small request batch of text, padded to its longest sentence: token ids in, embedding, masked encoder
        {"name": "base_text_b8_s61", "kind": "encoder", "model": "base", "batch": 8, "seq": 61, "input": "text", "graph": False},
        # a corner of the paper's latency grid: the larger model at sequence length 256, batch 4
        {"name": "large_b4_s256_graph", "kind": "encoder", "model": "large", "batch": 4, "seq": 256, "input": "activations", "graph": True},
        # the headline workload of bench.py
        {"name": "base_b32_graph", "kind": "encoder", "model": "base", "batch": 32, "seq": 128, "input": "activations", "graph": True},
        # longer text with a batch and a length that divide by nothing
        {"name": "base_text_b61_s251", "kind": "encoder", "model": "base", "batch": 61, "seq": 251, "input": "text", "graph": False},
        # long documents at full length
        {"name": "base_b64_s512", "kind": "encoder", "model": "base", "batch": 64, "seq": 512, "input": "activations", "graph": False},
        # throughput serving of the larger model: a padded batch, and the largest one
        {"name": "large_text_b32_s128", "kind": "encoder", "model": "large", "batch": 32, "seq": 128, "input": "text", "graph": False},
        {"name": "large_b256_s128", "kind": "encoder", "model": "large", "batch": 256, "seq": 128, "input": "activations", "graph": False},
        # an FFN block composed from the primitives over packed tokens (no padding, the sum of the sentence lengths)
        {"name": "ffn_base_t2741", "kind": "ffn", "model": "base", "tokens": 2741},
        # the three non-linear kernels on INT32 inputs, for a program with MatMuls of its own: Base activations, batch 32
        {"name": "nonlinear_base_b32", "kind": "nonlinear", "model": "base", "batch": 32, "seq": 128},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choices(["encoder", "layer", "ffn", "nonlinear"], [6, 1, 2, 1])[0]
    if kind == "layer":                      # at most what the static workspace holds (7 Base sequences of 128)
        model = rng.choice(["tiny", "base"])
        seq = _log_int(rng, 16, 200)
        return {"kind": kind, "model": model, "batch": _log_int(rng, 1, max(1, 800 // seq)), "seq": seq}
    model = rng.choice(["base", "large"])
    if kind == "ffn":
        return {"kind": kind, "model": model, "tokens": _log_int(rng, 32, MAX_TOKENS)}
    # half of the lengths are the powers of two that a fixed-shape program pads to, half are as the text has it
    seq = rng.choice([128, 256, 512]) if rng.random() < 0.5 else _log_int(rng, 16, MAX_SEQ)
    most = 8192 if kind == "nonlinear" else MAX_TOKENS * 3 // 4 if model == "large" and seq > 128 else MAX_TOKENS
    batch = max(1, _log_int(rng, seq, most) // seq)
    if kind == "nonlinear":
        return {"kind": kind, "model": model, "batch": batch, "seq": seq}
    return {"kind": kind, "model": model, "batch": batch, "seq": seq, "input": rng.choice(["activations", "text"]),
            "graph": batch * seq <= 4096 and rng.random() < 0.5}


# ---------------------------------------------------------------------------------------------- parameters
def _upload(a, dtype, dev):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=dtype)).to(dev)


def _i8(gen, *shape):
    return torch.randint(-127, 128, shape, dtype=torch.int8, device=gen.device, generator=gen)


def _activations(gen, tokens, hidden):
    """N(0, 1) activations at the scale of a LayerNorm output, symmetric INT8."""
    x = torch.randn(tokens, hidden, device=gen.device, generator=gen)
    return (x / S_ACT).round_().clamp_(-127, 127).to(torch.int8)


class _Linear:
    """INT8 weight [N, K] with bias and per-channel requantization; `out` = one (columns, S_out) per block of columns."""

    def __init__(self, gen, rng, n_in, S_in, *out):
        n = sum(c for c, _ in out)
        sw = np.exp(rng.normal(math.log(0.01), 0.3, size=n))
        self.w = _i8(gen, n, n_in)
        self.b = _upload(rng.integers(-(1 << 15), (1 << 15) + 1, size=n), np.int32, gen.device)
        at, mult, shift = 0, [], []
        for c, S_out in out:
            m, s = B.ibert_channel_dyadics_from_scales(S_in, sw[at:at + c], S_out)
            mult.append(m)
            shift.append(s)
            at += c
        self.m, self.s = _upload(np.concatenate(mult), np.int32, gen.device), _upload(np.concatenate(shift), np.int32, gen.device)


class _Norm:
    def __init__(self, gen, rng, hidden, S_out):
        g, b, self.shift = B.ibert_layernorm_params_from_float(rng.normal(1.0, 0.1, hidden), rng.normal(0.0, 0.1, hidden), S_out)
        self.g, self.b = _upload(g, np.int32, gen.device), _upload(b, np.int32, gen.device)


class _Layer:
    def __init__(self, gen, rng, hidden, heads, ffn, seq, sc):
        H = hidden
        self.parts = {"qkv": _Linear(gen, rng, H, sc["S_x"], (H, sc["S_q"]), (H, sc["S_k"]), (H, sc["S_v"])),
                      "o": _Linear(gen, rng, H, sc["S_ctx"], (H, sc["S_r1"])),
                      "1": _Linear(gen, rng, H, sc["S_h1"], (ffn, sc["S_g_in"])),
                      "2": _Linear(gen, rng, ffn, sc["S_g_out"], (H, sc["S_r2"]))}
        self.ln1, self.ln2 = _Norm(gen, rng, H, sc["S_h1"]), _Norm(gen, rng, H, sc["S_y"])
        w = B.LayerWeights()
        for k, p in self.parts.items():
            for f in "wbms":
                setattr(w, f + "_" + k, getattr(p, f).data_ptr())
        w.ln1_gamma_q, w.ln1_beta_q = self.ln1.g.data_ptr(), self.ln1.b.data_ptr()
        w.ln2_gamma_q, w.ln2_beta_q = self.ln2.g.data_ptr(), self.ln2.b.data_ptr()
        self.weights = w
        self.quant = B.ibert_layer_quant_from_scales(sc, seq, H // heads)
        self.quant.ln1_shift, self.quant.ln2_shift = self.ln1.shift, self.ln2.shift


def _scales(model, batch, seq):
    hidden, heads, ffn, layers = MODELS[model]
    cfg = synth.EncoderConfig(model, hidden, heads, ffn, seq, batch, layers)
    return synth.model_scales(cfg, S_ACT)


# ---------------------------------------------------------------------------------------------- states
class _Encoder:
    """All layers, the workspace and the input; with text, the embedding tables, token ids and sentence lengths."""

    def __init__(self, case, gen, rng):
        self.hidden, self.heads, self.ffn, self.n = MODELS[case["model"]]
        self.batch, self.seq, self.single = case["batch"], case["seq"], case["kind"] == "layer"
        scales = _scales(case["model"], self.batch, self.seq)[:1 if self.single else self.n]
        self.layers = [_Layer(gen, rng, self.hidden, self.heads, self.ffn, self.seq, sc) for sc in scales]
        self.weights = (B.LayerWeights * len(self.layers))(*[l.weights for l in self.layers])
        self.quant = (B.LayerQuant * len(self.layers))(*[l.quant for l in self.layers])
        tokens = self.batch * self.seq
        self.x = _activations(gen, tokens, self.hidden)
        self.y = torch.empty_like(self.x)
        self.lens = None
        self.text = case.get("input") == "text"
        if self.text:
            self.lens = _upload(synth.key_lengths(self.batch, self.seq, seed=int(rng.integers(1 << 30))), np.int32, gen.device)
            self.ids = _upload((rng.zipf(1.3, size=tokens) - 1) % VOCAB, np.int32, gen.device)
            tok, pos = (torch.randn(n, self.hidden, device=gen.device, generator=gen) * std for n, std in ((VOCAB, 0.05), (MAX_SEQ, 0.02)))
            S_tok, S_pos, S_r = float(tok.abs().max()) / 127, float(pos.abs().max()) / 127, 2.0 ** -12
            self.tok, self.pos = ((t / s).round_().clamp_(-127, 127).to(torch.int8) for t, s in ((tok, S_tok), (pos, S_pos)))
            self.tok_dy, self.pos_dy = B.ibert_dyadic_from_double(S_tok / S_r), B.ibert_dyadic_from_double(S_pos / S_r)
            self.emb_ln = _Norm(gen, rng, self.hidden, S_ACT)
        shape = (self.batch, self.seq, self.hidden, self.heads, self.ffn)
        self.ws = None
        if not self.single:
            self.ws = torch.empty(B.ibert_encoder_workspace_bytes(*shape), dtype=torch.uint8, device=gen.device)
        elif case["model"] == "tiny":        # (the Base layer runs in the library's own workspace)
            self.ws = torch.empty(B.ibert_encoder_layer_workspace_bytes(*shape), dtype=torch.uint8, device=gen.device)
        self.graph = None
        if case.get("graph"):
            self.call()
            torch.cuda.synchronize()
            self.graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(self.graph):
                self.call()

    def call(self):
        shape = (self.batch, self.seq, self.hidden, self.heads, self.ffn)
        if self.text:
            B.ibert_embedding_i(self.ids, self.tok, self.pos, self.batch * self.seq, self.seq, self.hidden, VOCAB, MAX_SEQ,
                                self.tok_dy, self.pos_dy, self.emb_ln.g, self.emb_ln.b, self.emb_ln.shift, self.x, self.hidden)
        if self.single and self.ws is None:
            B.ibert_encoder_layer_static_i(self.weights[0], self.quant[0], self.x, self.y, *shape)
        elif self.single:
            B.ibert_encoder_layer_i(self.weights[0], self.quant[0], self.x, self.y, *shape, self.ws)
        elif self.text:
            B.ibert_encoder_masked_i(self.weights, self.quant, self.n, self.x, self.y, *shape, self.lens, self.ws)
        else:
            B.ibert_encoder_i(self.weights, self.quant, self.n, self.x, self.y, *shape, self.ws)

    def run(self):
        if self.graph is not None:
            self.graph.replay()
        else:
            self.call()
        return self.y


class _Ffn:
    """h -> LayerNorm(W_2 GELU(W_1 h) + h) over packed tokens, from the primitives."""

    def __init__(self, case, gen, rng):
        self.hidden, _, self.ffn, _ = MODELS[case["model"]]
        self.tokens = T = case["tokens"]
        sc = _scales(case["model"], 1, T)[0]
        self.up = _Linear(gen, rng, self.hidden, S_ACT, (self.ffn, sc["S_g_in"]))
        self.down = _Linear(gen, rng, self.ffn, sc["S_g_out"], (self.hidden, sc["S_r2"]))
        self.ln = _Norm(gen, rng, self.hidden, sc["S_y"])
        self.gelu = B.ibert_gelu_params_from_scale(sc["S_g_in"], sc["S_g_out"])
        self.h = _activations(gen, T, self.hidden)
        self.g = torch.empty(T, self.ffn, dtype=torch.int8, device=gen.device)
        self.scratch = torch.empty(T, self.ffn, dtype=torch.int32, device=gen.device)
        self.r = torch.empty(T, self.hidden, dtype=torch.int16, device=gen.device)
        self.y = torch.empty_like(self.h)

        def desc(n, k, out_dtype, clamp):
            d = B.GemmDesc()
            d.M, d.N, d.K, d.batch_outer, d.batch_inner = T, n, k, 1, 1
            d.lda, d.ldw, d.ldc, d.ldr = k, k, n, n
            d.per_channel, d.out_dtype, d.out_clamp = 1, out_dtype, clamp
            return d
        self.d_up = desc(self.ffn, self.hidden, B.I8, 127)
        self.d_down = desc(self.hidden, self.ffn, B.I16, 32767)
        self.d_down.residual_dy = B.ibert_dyadic_from_double(sc["S_h1"] / sc["S_r2"])

    def run(self):
        u, d, H = self.up, self.down, self.hidden
        B.ibert_gemm_i8_gelu(self.d_up, self.h, u.w, u.b, u.m, u.s, self.gelu, self.g, self.scratch)
        B.ibert_gemm_i8_requant(self.d_down, self.g, d.w, d.b, d.m, d.s, self.h, self.r)
        B.ibert_layernorm_i16(self.r, self.y, self.tokens, H, H, H, self.ln.g, self.ln.b, self.ln.shift)
        return self.g, self.r, self.y


class _NonLinear:
    """Softmax over the attention logits, GELU over the FFN activation and LayerNorm over the hidden states of a batch."""

    def __init__(self, case, gen, rng):
        self.hidden, heads, ffn, _ = MODELS[case["model"]]
        self.cols, self.tokens = case["seq"], case["batch"] * case["seq"]
        self.rows = heads * self.tokens

        def normal(rows, cols, std, scale):
            return (torch.randn(rows, cols, device=gen.device, generator=gen) * (std / scale)).round_().to(torch.int32)
        self.sx, self.gx = normal(self.rows, self.cols, 4.0, 2.0 ** -6), normal(self.tokens, ffn, 2.0, 2.0 ** -7)
        self.lx = normal(self.tokens, self.hidden, 3.0, 2.0 ** -8)
        self.sy, self.gy, self.ly = (torch.empty(t.shape, dtype=torch.int8, device=gen.device) for t in (self.sx, self.gx, self.lx))
        self.sp = B.ibert_softmax_params_from_scale(2.0 ** -6, self.cols)
        self.gp = B.ibert_gelu_params_from_scale(2.0 ** -7, 8.0 / 127)
        self.ln = _Norm(gen, rng, self.hidden, S_ACT)

    def run(self):
        L, H = self.cols, self.hidden
        B.ibert_softmax_i(self.sx, self.sy, self.rows, L, L, L, self.sp)
        B.ibert_gelu_i(self.gx, self.gy, self.gx.numel(), self.gp)
        B.ibert_layernorm_i(self.lx, self.ly, self.tokens, H, H, H, self.ln.g, self.ln.b, self.ln.shift)
        return self.sy, self.gy, self.ly


_KINDS = {"encoder": _Encoder, "layer": _Encoder, "ffn": _Ffn, "nonlinear": _NonLinear}


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return _KINDS[case["kind"]](case, gen, np.random.default_rng([synth.SEED, seed]))


def run(state):
    return state.run()


# ---------------------------------------------------------------------------------------------- what a pass takes
def work(case):
    H, heads, F, layers = MODELS[case["model"]]
    if case["kind"] == "ffn":
        T = case["tokens"]
        return {"bytes": 2 * H * F + 12 * (H + F) + 8 * H + T * (H + F + 2 * H + H), "flops": 4 * T * H * F}
    B_, L = case["batch"], case["seq"]
    T = B_ * L
    if case["kind"] == "nonlinear":
        n = heads * T * L + T * F + T * H
        return {"bytes": 5 * n + 8 * H, "flops": 12 * n}
    layers = 1 if case["kind"] == "layer" else layers
    text = case.get("input") == "text"
    keys = 0.625 * L if text else L          # sentence lengths are uniform in [L/4, L]; masked keys need no work
    per_layer = 2 * T * (4 * H * H + 2 * H * F) + 4 * T * keys * H
    weights = layers * (4 * H * H + 2 * H * F + 12 * (5 * H + F) + 16 * H)
    table = T * (4 + H) + L * H if text else T * H
    return {"bytes": weights + table + T * H, "flops": layers * per_layer}


def tolerance(case):
    return "exact"
