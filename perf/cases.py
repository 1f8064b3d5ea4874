"""The work by which this library's speed is judged: what a program that runs HGF models has it do,
through the public entry points, from the smallest call to the largest.

Shapes are those of the benchmark configurations (paper_2602_05269_amd.synth.CONFIGS) and of the
block test (the paper's own model: d = 512, 8 heads, MLP width 1365, context 512).  A case is a dict
of plain values; `listed()` names twelve, `draw(rng)` makes more of the same kinds:

  linear     one hgf_linear_forward                             (a layer on its own)
  stack      a layer list through hgf_stack_forward             (decode and prefill of a model's linears)
  mlp        hgf_swiglu_forward, then the down projection       (the model's gated MLP, block after block)
  block      one decode step of a whole block                   (LayerNorm q, k, v; caches; attention; MLP)
  attention  hgf_diff_attention_decode                          (the step's attention alone, long caches)
  b3         hgf_linear_forward_b3                              (the 1.6-bit format at decode)
  pack       hgf_quantize_pack_weights[_b3]                     (loading a model: ternarise and pack)

Weights are drawn with the fan-in deviation 1.5 / sqrt(d_in), with which a ternarised layer keeps the
magnitude of its input (as the norms of a trained model would), activations with the heavy tails of
the benchmark configurations.

Every linear quantises its input to 8 bits with one scale per token, so where two correct
implementations differ in the last bit of one layer's fp16 output, single codes of the next layer
flip, and the difference grows by about the quantiser's step with every further layer.  Layer lists
are therefore chained over four dependent groups of layers (one whole block of q, k, v, o, up, gate,
down; two blocks of up, gate, down) and then read a fresh input, as a block's linears do behind the
caller's residual and norm."""
from __future__ import annotations

import math

import torch

from paper_2602_05269_amd import binding as hb
from paper_2602_05269_amd import synth

# ------------------------------------------------------------------------------------- the cases


def listed():
    return [
        # the smallest call: one small layer for a handful of tokens (configuration 0), where the
        # launches and the host path are everything
        {"name": "linear_256_m8", "kind": "linear", "d_in": 256, "d_out": 256, "rank": 16, "tokens": 8,
         "act": "normal", "ln": False, "static": False},
        # one token through all linears of the paper's own model size (configuration 1): 14.7 MB of
        # weights in cache, a chain of latencies
        {"name": "stack_512_m1", "kind": "stack", "cfg": 1, "blocks": 8, "tokens": 1, "ln": False},
        # the headline: one token through 7B-shape FFN blocks (configuration 4), weights from HBM
        {"name": "stack_7b_m1", "kind": "stack", "cfg": 4, "blocks": 16, "tokens": 1, "ln": False},
        # decode for a batch of eight users, the same shapes (configuration 4)
        {"name": "stack_7b_m8", "kind": "stack", "cfg": 4, "blocks": 8, "tokens": 8, "ln": False},
        # decode for sixteen users through whole 1.2B-shape layers (configuration 2)
        {"name": "stack_1b_m16", "kind": "stack", "cfg": 2, "blocks": 12, "tokens": 16, "ln": False},
        # the gated MLP at the largest decode batch of configuration 4
        {"name": "mlp_7b_m64", "kind": "mlp", "d": 4096, "ffn": 11008, "rank": 128, "blocks": 8, "tokens": 64},
        # reading a prompt of a ragged 500 tokens with the paper's model and its LayerNorms
        {"name": "stack_512_ln_m500", "kind": "stack", "cfg": 1, "blocks": 4, "tokens": 500, "ln": True},
        # a long prompt through a 3B-shape block (configuration 3): the largest
        {"name": "stack_3b_m2048", "kind": "stack", "cfg": 3, "blocks": 1, "tokens": 2048, "ln": False},
        # one decode step of a whole block of the paper's model for 24 sequences of ragged lengths
        {"name": "block_512_b24", "kind": "block", "d": 512, "heads": 8, "hidden": 1365, "rank": 16, "sequences": 24,
         "context": 512},
        # attention over long ragged caches, 7B shape
        {"name": "attention_7b_b8", "kind": "attention", "sequences": 8, "context": 4096, "heads": 32, "d_h": 64},
        # the 1.6-bit format: the 7B-shape up projections of twenty blocks, one token
        {"name": "b3_7b_m1", "kind": "b3", "d_in": 4096, "d_out": 11008, "rank": 128, "layers": 20, "tokens": 1},
        # loading a model: one 7B-shape matrix from its fp32 latents to packed codes
        {"name": "pack_7b", "kind": "pack", "d_in": 4096, "d_out": 11008, "format": "2bit"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# the most that one drawn case may do (a little under the largest listed ones)
_MOST_FLOPS, _MOST_BYTES = 4.6e11, 7.0e8


def draw(rng):
    while True:
        case = _draw(rng)
        w = work(case)
        if w["flops"] <= _MOST_FLOPS and w["bytes"] <= _MOST_BYTES:
            return case


def _draw(rng):
    kind = rng.choice(["linear", "stack", "stack", "stack", "mlp", "block", "attention", "b3", "pack"])
    odd = lambda v: v if rng.random() < 0.5 else v | 1
    if kind == "linear":
        return {"kind": kind, "d_in": odd(_log(rng, 64, 8192)), "d_out": odd(_log(rng, 64, 8192)),
                "rank": rng.choice([0, 8, 16, 24, 32, 64, 100, 128]), "tokens": _log(rng, 1, 2048),
                "act": rng.choice(["normal", "student_t3", "student_t4"]), "ln": rng.random() < 0.3,
                "static": rng.random() < 0.2}
    if kind == "stack":
        cfg = rng.choice([1, 2, 3, 4])
        few = rng.random() < 0.6
        tokens = _log(rng, 1, 64) if few else _log(rng, 65, 2048)
        blocks = {1: 8, 2: 12, 3: 8, 4: 8}[cfg] if few else {1: 4, 2: 2, 3: 1, 4: 1}[cfg]
        return {"kind": kind, "cfg": cfg, "blocks": rng.randint(max(1, blocks // 2), blocks), "tokens": tokens,
                "ln": rng.random() < 0.25}
    if kind == "mlp":
        d, ffn, rank = rng.choice([(512, 1365, 16), (2048, 8192, 64), (3072, 8192, 64), (4096, 11008, 128)])
        tokens = _log(rng, 1, 1024)
        return {"kind": kind, "d": d, "ffn": ffn, "rank": rank, "blocks": 8 if tokens <= 64 else 1, "tokens": tokens}
    if kind == "block":
        d, heads, hidden, rank, ctx = rng.choice([(512, 8, 1365, 16, 512), (512, 4, 1365, 32, 512), (2048, 16, 8192, 64, 1024)])
        return {"kind": kind, "d": d, "heads": heads, "hidden": hidden, "rank": rank, "sequences": _log(rng, 1, 64),
                "context": ctx}
    if kind == "attention":
        d_h = rng.choice([32, 64, 128])
        return {"kind": kind, "sequences": _log(rng, 1, 64), "context": _log(rng, 64, 8192),
                "heads": rng.choice([4, 8, 16, 32]), "d_h": d_h}
    if kind == "b3":
        d_in, d_out, rank = rng.choice([(512, 2048, 32), (2048, 8192, 64), (4096, 11008, 128), (11008, 4096, 128),
                                        (4095, 1365, 32)])
        return {"kind": kind, "d_in": d_in, "d_out": d_out, "rank": rank, "layers": rng.randint(4, 20),
                "tokens": rng.randint(1, 4 if d_in < 8192 else 2)}
    return {"kind": kind, "d_in": odd(_log(rng, 256, 11008)), "d_out": odd(_log(rng, 256, 11008)),
            "format": rng.choice(["2bit", "b3"])}


# ------------------------------------------------------------------------------------- their inputs


class _Maker:
    """Seeded tensors on the GPU."""

    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(seed)

    def normal(self, *shape):
        return torch.randn(shape, generator=self.gen, device="cuda")

    def activations(self, kind, M, K):
        """fp16 [M, K] of one of the distributions of synth.draw_activations."""
        x = self.normal(M, K)
        if kind == "outlier":                       # one channel in a hundred is twenty times as large
            chans = torch.randperm(K, generator=self.gen, device="cuda")[:math.ceil(0.01 * K)]
            x[:, chans] *= 20.0
        elif kind.startswith("student_t"):          # normal / sqrt(chi^2 / nu)
            nu = int(kind[-1])
            chi2 = sum(self.normal(M, K) ** 2 for _ in range(nu))
            x = x * torch.rsqrt(chi2 / nu)
        return x.clamp(-synth.FP16_MAX, synth.FP16_MAX).half()

    def latent(self, d_in, d_out, rank, ln=False, lora_std=0.02):
        """One linear before it is ternarised: W, (A, B, alpha) or None, LayerNorm parameters."""
        W = self.normal(d_out, d_in) * (1.5 / math.sqrt(d_in))
        low = None
        if rank:
            low = ((self.normal(rank, d_in) * lora_std).half(), (self.normal(d_out, rank) * lora_std).half(),
                   self.normal(d_out).half())
        norm = {}
        if ln:
            norm = {"ln_gamma": 1.0 + 0.25 * self.normal(d_in), "ln_beta": 0.2 * self.normal(d_in)}
        return W, low, norm

    def layer(self, d_in, d_out, rank, ws, src=0, dst=1, ln=False, lora_std=0.02, b3=False):
        W, low, norm = self.latent(d_in, d_out, rank, ln, lora_std)
        A, B, alpha = low or (None, None, None)
        if b3:
            packed, s_w = hb.hgf_quantize_pack_weights_b3(W, ws)
            return hb.Layer(packed, s_w, d_out, d_in, A, B, alpha)
        return hb.Layer.from_latent(W, A, B, alpha, ws, src_slot=src, dst_slot=dst, **norm)


def _wiring(case):
    """(projection, source slot, destination slot) of every linear, and the slots that hold inputs.
    A block's linears as synth.stack_wiring has them; a new input after every `chain` blocks."""
    chain = 2 if case["cfg"] == 4 else 1
    out, inputs, free, block_in = [], [], 0, 0
    for b in range(case["blocks"]):
        if b % chain == 0:
            block_in, free = free, free + 1
            inputs.append(block_in)
        at = {}
        for p in synth.CONFIGS[case["cfg"]].projections:
            src = block_in
            if p.name == "o":
                src = at["v"]
            elif p.name in ("up", "gate"):
                src = at.get("o", block_in)
            elif p.name == "down":
                src = at["up"]
            at[p.name], free = free, free + 1
            out.append((p, src, at[p.name]))
        block_in = at["down"]
    return out, inputs


def _lengths(case):
    """Ragged cache lengths, from a full cache down: the same for every seed."""
    B, L = case["sequences"], case["context"]
    return [L if b == 0 else 1 + (b * 2654435761 % 4294967296) * (L - 1) // 4294967296 for b in range(B)]


def prepare(case, seed):
    mk, kind = _Maker(seed), case["kind"]
    if kind == "linear":
        M, K, N, r = case["tokens"], case["d_in"], case["d_out"], case["rank"]
        ws = hb.Workspace(M, K, N, r)
        # (the entry point with the library's own fixed scratch takes what fits that scratch)
        static = case["static"] and hb.hgf_static_scratch_needed(M, K, N, r) <= hb.hgf_static_scratch_bytes()
        return {"kind": "static" if static else kind, "ws": ws, "layer": mk.layer(K, N, r, ws, ln=case["ln"]),
                "x": mk.activations(case["act"], M, K), "y": torch.empty((M, N), dtype=torch.float16, device="cuda")}
    if kind == "stack":
        c, M = synth.CONFIGS[case["cfg"]], case["tokens"]
        wide = max(max(p.d_in, p.d_out) for p in c.projections)
        ws = hb.Workspace(M, wide, wide, c.rank)
        wiring, inputs = _wiring(case)
        slots = [None] * (1 + max(dst for _, _, dst in wiring))
        for s in inputs:
            slots[s] = mk.activations(c.act, M, wiring[0][0].d_in)
        layers, outs = [], []
        for i, (p, src, dst) in enumerate(wiring):
            if i % len(c.projections) == 0:         # a block's outputs lie in one buffer, one after the other
                outs.append(torch.empty(M * sum(q.d_out for q in c.projections), dtype=torch.float16, device="cuda"))
                at = 0
            layers.append(mk.layer(p.d_in, p.d_out, c.rank, ws, src, dst, case["ln"], c.lora_std))
            slots[dst] = outs[-1][at:at + M * p.d_out].view(M, p.d_out)
            at += M * p.d_out
        return {"kind": kind, "ws": ws, "stack": hb.Stack(layers, slots, M), "outs": outs}
    if kind == "mlp":
        M, d, ffn, r = case["tokens"], case["d"], case["ffn"], case["rank"]
        ws = hb.Workspace(M, max(d, ffn), max(d, ffn), r)
        half = lambda n: torch.empty((M, n), dtype=torch.float16, device="cuda")
        return {"kind": kind, "ws": ws, "blocks": [
            {"x": mk.activations("student_t3", M, d), "gate": mk.layer(d, ffn, r, ws), "up": mk.layer(d, ffn, r, ws),
             "down": mk.layer(ffn, d, r, ws), "z": half(ffn), "y": half(d)} for _ in range(case["blocks"])]}
    if kind == "block":
        B, L, H, d, hid, r = (case[k] for k in ("sequences", "context", "heads", "d", "hidden", "rank"))
        dh = d // (2 * H)
        ws = hb.Workspace(B, max(d, hid), max(d, hid), r)
        lens = _lengths(case)
        return {"kind": kind, "ws": ws, "B": B, "H": H, "dh": dh, "x": mk.activations("student_t4", B, d),
                "q": mk.layer(d, d, r, ws, ln=True), "k": mk.layer(d, d, r, ws, ln=True), "v": mk.layer(d, d // 2, r, ws, ln=True),
                "o": mk.layer(d // 2, d, 0, ws), "gate": mk.layer(d, hid, r, ws), "up": mk.layer(d, hid, r, ws),
                "down": mk.layer(hid, d, r, ws),
                "k_cache": mk.normal(B, L, 2 * H, dh).half(), "v_cache": mk.normal(B, L, H, dh).half(),
                "lens": torch.tensor(lens, dtype=torch.int32, device="cuda"),
                "rows": torch.tensor([b * L + n - 1 for b, n in enumerate(lens)], device="cuda"),
                "scratch": torch.empty(hb.lib().hgf_diff_attention_workspace_bytes(B, L, H, dh), dtype=torch.uint8, device="cuda")}
    if kind == "attention":
        B, L, H, dh = (case[k] for k in ("sequences", "context", "heads", "d_h"))
        return {"kind": kind, "q": mk.normal(B, 2 * H, dh).half(), "k": mk.normal(B, L, 2 * H, dh).half(),
                "v": mk.normal(B, L, H, dh).half(), "lens": torch.tensor(_lengths(case), dtype=torch.int32, device="cuda"),
                "out": torch.empty((B, H, dh), dtype=torch.float16, device="cuda"),
                "scratch": torch.empty(hb.lib().hgf_diff_attention_workspace_bytes(B, L, H, dh), dtype=torch.uint8, device="cuda")}
    if kind == "b3":
        M, K, N, r = case["tokens"], case["d_in"], case["d_out"], case["rank"]
        ws = hb.Workspace(M, K, N, r)
        return {"kind": kind, "ws": ws, "layers": [
            {"layer": mk.layer(K, N, r, ws, b3=True), "x": mk.activations("student_t3", M, K),
             "y": torch.empty((M, N), dtype=torch.float16, device="cuda")} for _ in range(case["layers"])]}
    K, N = case["d_in"], case["d_out"]
    return {"kind": "pack_" + case["format"], "ws": hb.Workspace(1, K, N, 0), "W": mk.normal(N, K) * (1.5 / math.sqrt(K))}


# ------------------------------------------------------------------------------------- one pass


def run(s):
    kind = s["kind"]
    if kind == "linear":
        return hb.hgf_linear_forward(s["x"], s["layer"], s["ws"], y=s["y"])
    if kind == "static":
        return hb.hgf_linear_forward_static(s["x"], s["layer"], s["y"])
    if kind == "stack":
        hb.hgf_stack_forward(s["stack"], s["ws"])
        return s["outs"]
    if kind == "mlp":
        for b in s["blocks"]:
            hb.hgf_swiglu_forward(b["x"], b["gate"], b["up"], s["ws"], z=b["z"])
            hb.hgf_linear_forward(b["z"], b["down"], s["ws"], y=b["y"])
        return [t for b in s["blocks"] for t in (b["z"], b["y"])]
    if kind == "block":
        ws, x, B, H, dh = s["ws"], s["x"], s["B"], s["H"], s["dh"]
        q = hb.hgf_linear_forward(x, s["q"], ws)
        k = hb.hgf_linear_forward(x, s["k"], ws)
        v = hb.hgf_linear_forward(x, s["v"], ws)
        s["k_cache"].view(-1, 2 * H * dh).index_copy_(0, s["rows"], k)
        s["v_cache"].view(-1, H * dh).index_copy_(0, s["rows"], v)
        a = hb.hgf_diff_attention_decode(q.view(B, 2 * H, dh), s["k_cache"], s["v_cache"], s["lens"], 0.8, workspace=s["scratch"])
        x1 = x + hb.hgf_linear_forward(a.view(B, H * dh), s["o"], ws)
        z = hb.hgf_swiglu_forward(x1, s["gate"], s["up"], ws)
        x2 = x1 + hb.hgf_linear_forward(z, s["down"], ws)
        return {"out": x2, "k": k, "v": v}
    if kind == "attention":
        return hb.hgf_diff_attention_decode(s["q"], s["k"], s["v"], s["lens"], 0.8, out=s["out"], workspace=s["scratch"])
    if kind == "b3":
        return [hb.hgf_linear_forward_b3(l["x"], l["layer"], s["ws"], y=l["y"]) for l in s["layers"]]
    if kind == "pack_2bit":
        return hb.hgf_quantize_pack_weights(s["W"], s["ws"])
    return hb.hgf_quantize_pack_weights_b3(s["W"], s["ws"])


# ------------------------------------------------------------------------------------- what a pass needs


def _linear_work(M, K, N, r, ln=False, x_in=True, y_out=True, bits=2.0):
    """Packed weights, A, B, gate, LayerNorm parameters, x and y once; the integer contraction and
    the two low-rank products."""
    nbytes = K * N * bits / 8 + (2 * r * (K + N) + 2 * N if r else 0) + 4 + (8 * K if ln else 0)
    return nbytes + 2 * M * K * x_in + 2 * M * N * y_out, 2.0 * M * K * N + 2.0 * M * r * (K + N)


def _attention_work(case, H, dh):
    n = sum(_lengths(case))
    B = case["sequences"]
    return n * 3 * H * dh * 2 + B * (2 * H + H) * dh * 2, n * H * dh * (4 + 4.0)


def work(case):
    kind = case["kind"]
    if kind == "linear":
        b, f = _linear_work(case["tokens"], case["d_in"], case["d_out"], case["rank"], case["ln"])
    elif kind == "stack":
        r, M = synth.CONFIGS[case["cfg"]].rank, case["tokens"]
        parts, seen = [], set()
        for p, src, _ in _wiring(case)[0]:          # (layers that share an input read it once)
            parts.append(_linear_work(M, p.d_in, p.d_out, r, case["ln"], x_in=src not in seen))
            seen.add(src)
        b, f = (sum(v) for v in zip(*parts))
    elif kind == "mlp":
        M, d, ffn, r = case["tokens"], case["d"], case["ffn"], case["rank"]
        parts = [_linear_work(M, d, ffn, r, y_out=False), _linear_work(M, d, ffn, r, x_in=False), _linear_work(M, ffn, d, r)]
        b, f = (case["blocks"] * sum(v) for v in zip(*parts))
    elif kind == "block":
        M, d, hid, r = case["sequences"], case["d"], case["hidden"], case["rank"]
        parts = [_linear_work(M, d, d, r, True), _linear_work(M, d, d, r, True, x_in=False),
                 _linear_work(M, d, d // 2, r, True, x_in=False), _attention_work(case, case["heads"], d // (2 * case["heads"])),
                 _linear_work(M, d // 2, d, 0), _linear_work(M, d, hid, r, y_out=False), _linear_work(M, d, hid, r, x_in=False),
                 _linear_work(M, hid, d, r)]
        b, f = (sum(v) for v in zip(*parts))
    elif kind == "attention":
        b, f = _attention_work(case, case["heads"], case["d_h"])
    elif kind == "b3":
        b, f = _linear_work(case["tokens"], case["d_in"], case["d_out"], case["rank"], bits=1.6)
        b, f = b * case["layers"], f * case["layers"]
    else:
        n = case["d_in"] * case["d_out"]
        b, f = n * (4 + (0.25 if case["format"] == "2bit" else 0.2)), 3.0 * n
    return {"bytes": float(b), "flops": float(f)}


def tolerance(case):
    """About four times the largest difference measured between the library and the same path in 64
    bits (exact integers, fp64 sums, fp16 where the library's results are fp16): 1.5e-4 for one
    linear (two fp16 roundings: SiLU(A x), y), 1.8e-5 for the attention step.  Where an output feeds
    another linear, elements that moved to the neighbouring fp16 number flip codes of its quantiser
    (see above): 1.9e-3 behind one linear, 7.1e-3 behind three."""
    kind = case["kind"]
    if kind == "pack":
        return "exact"
    if kind in ("stack", "block"):
        return {"rel": 3e-2, "max": 0.3}
    if kind == "mlp":
        return {"rel": 8e-3, "max": 0.15}
    if kind == "attention":
        return {"rel": 1e-4, "max": 4e-3}
    return {"rel": 6e-4, "max": 5e-3}


# ------------------------------------------------------------------------------------- the same in 64 bits


def _scale_of(W):
    return W.double().abs().mean().clamp_min(1e-5).float()


def _norm64(x, norm):
    """The row that is quantised: LayerNorm by its definition (fp64 reductions, fp32 elementwise)."""
    if not norm:
        return x.float()
    mean = x.double().mean(1, keepdim=True)
    var = ((x.double() - mean) ** 2).mean(1, keepdim=True)
    return ((x.float() - mean.float()) * (1.0 / torch.sqrt(var + 1e-5)).float()) * norm["ln_gamma"] + norm["ln_beta"]


def _linear64(x, latent):
    """fp64 outputs of one linear for fp16 tokens: the codes are whole numbers that the definition
    fixes (fp32 scale, round half to even), everything behind them is in 64 bits."""
    W, low, norm = latent
    s_w = _scale_of(W)
    T = torch.round(W * (1.0 / s_w)).clamp(-1, 1).double()
    v = _norm64(x, norm)
    amax = v.abs().amax(1, keepdim=True).clamp_min(1e-5)
    codes = torch.round(v * (127.0 / amax)).clamp(-127, 127)
    y = (codes.double() @ T.t()) * (amax.double() / 127.0) * s_w.double()
    if low:
        A, B, alpha = (t.double() for t in low)
        y += torch.tanh(alpha) * (torch.nn.functional.silu(x.double() @ A.t()) @ B.t())
    return y


def _attention64(q, k, v, lens, lam):
    """[B, H, d_h] fp64 of the differential attention step; q [B, 2H, d_h], caches [B, L, heads, d_h]."""
    lam = float(torch.tensor(lam, dtype=torch.float32))
    H = v.shape[2]
    out = []
    for b, n in enumerate(lens):
        s = (k[b, :n].double() * q[b].double()).sum(-1) / math.sqrt(q.shape[2])
        p = torch.softmax(s, 0)
        out.append(0.5 * ((p[:, :H] - lam * p[:, H:]).unsqueeze(-1) * v[b, :n].double()).sum(0))
    return torch.stack(out)


def exact(case, seed):
    """What run() returns for these inputs, from torch in 64 bits: the tensors are drawn in the order
    of prepare(), results that another entry point reads are rounded to fp16 as its interface says,
    and the outputs themselves are not rounded."""
    mk, kind = _Maker(seed), case["kind"]
    if kind == "linear":
        M, K, N, r = case["tokens"], case["d_in"], case["d_out"], case["rank"]
        lat = mk.latent(K, N, r, case["ln"])
        return _linear64(mk.activations(case["act"], M, K), lat)
    if kind == "stack":
        c, M = synth.CONFIGS[case["cfg"]], case["tokens"]
        wiring, inputs = _wiring(case)
        slots = {s: mk.activations(c.act, M, wiring[0][0].d_in) for s in inputs}
        outs = []
        for i, (p, src, dst) in enumerate(wiring):
            if i % len(c.projections) == 0:
                outs.append([])
            y = _linear64(slots[src], mk.latent(p.d_in, p.d_out, c.rank, case["ln"], c.lora_std))
            slots[dst] = y.half()
            outs[-1].append(y.flatten())
        return [torch.cat(b) for b in outs]
    if kind == "mlp":
        M, d, ffn, r = case["tokens"], case["d"], case["ffn"], case["rank"]
        outs = []
        for _ in range(case["blocks"]):
            x = mk.activations("student_t3", M, d)
            z = torch.nn.functional.silu(_linear64(x, mk.latent(d, ffn, r))) * _linear64(x, mk.latent(d, ffn, r))
            outs += [z, _linear64(z.half(), mk.latent(ffn, d, r))]
        return outs
    if kind == "block":
        B, L, H, d, hid, r = (case[k] for k in ("sequences", "context", "heads", "d", "hidden", "rank"))
        dh = d // (2 * H)
        lens = _lengths(case)
        x = mk.activations("student_t4", B, d)
        q, k, v = (_linear64(x, mk.latent(d, n, r, True)) for n in (d, d, d // 2))
        o, gate, up, down = (mk.latent(*shape) for shape in ((d // 2, d, 0), (d, hid, r), (d, hid, r), (hid, d, r)))
        kc, vc = mk.normal(B, L, 2 * H, dh).half(), mk.normal(B, L, H, dh).half()
        for b, n in enumerate(lens):
            kc[b, n - 1], vc[b, n - 1] = k[b].half().view(2 * H, dh), v[b].half().view(H, dh)
        a = _attention64(q.half().view(B, 2 * H, dh), kc, vc, lens, 0.8).half().view(B, H * dh)
        x1 = (x.double() + _linear64(a, o)).half()
        z = (torch.nn.functional.silu(_linear64(x1, gate)) * _linear64(x1, up)).half()
        return {"out": x1.double() + _linear64(z, down), "k": k, "v": v}
    if kind == "attention":
        B, L, H, dh = (case[k] for k in ("sequences", "context", "heads", "d_h"))
        q, k, v = mk.normal(B, 2 * H, dh).half(), mk.normal(B, L, 2 * H, dh).half(), mk.normal(B, L, H, dh).half()
        return _attention64(q, k, v, _lengths(case), 0.8)
    if kind == "b3":
        M, K, N, r = case["tokens"], case["d_in"], case["d_out"], case["rank"]
        outs = []
        for _ in range(case["layers"]):
            lat = mk.latent(K, N, r)
            outs.append(_linear64(mk.activations("student_t3", M, K), lat))
        return outs
    W = mk.normal(case["d_out"], case["d_in"]) * (1.5 / math.sqrt(case["d_in"]))
    return (None, W.double().abs().mean().clamp_min(1e-5).view(1))     # (the codes: whole bytes, no rounding)
