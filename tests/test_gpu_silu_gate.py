"""SiLU and the gate are computed as exactly as fp32 allows, in every kernel that serves few tokens: layers whose
other terms are known exactly show the one function behind its fp16 rounding.  An output has to be the rounding of
some value within the function's fp32 error of the exact one: 2^-21 for the gate (two units in the last place of
tanh and its product's rounding, doubled), 2.4e-7 for SiLU (one unit of the exponential, the sum's and the
quotient's half units)."""
import numpy as np
import pytest
import torch

from paper_2602_05269_amd import binding as hb

pytestmark = pytest.mark.gpu


def _layer(K, N, rank, B0, alpha, ws, b3=False):
    """No weights; A picks column 0 for rank 0, whose row of B is B0: y = tanh(alpha) B0 SiLU(x[:, 0])."""
    pack = hb.hgf_quantize_pack_weights_b3 if b3 else hb.hgf_quantize_pack_weights
    packed, s_w = pack(torch.zeros((N, K), device="cuda"), ws)
    A = torch.zeros((rank, K), dtype=torch.float16, device="cuda")
    A[0, 0] = 1
    B = torch.zeros((N, rank), dtype=torch.float16, device="cuda")
    B[:, 0] = B0
    return hb.Layer(packed, s_w, N, K, A, B, alpha)


def _tokens(M, K, first):
    x = torch.zeros((M, K), dtype=torch.float16, device="cuda")
    x[:, 0] = first                          # 24 and more: SiLU(x) = x in fp32
    return x


def _assert_rounded(got, exact, rel):
    lo, hi = (exact - rel * np.abs(exact)).astype(np.float16), (exact + rel * np.abs(exact)).astype(np.float16)
    bad = ~((got >= lo) & (got <= hi))
    assert not bad.any(), f"{int(bad.sum())} of {bad.size}, the first {got[bad][0]!r} for {exact[bad][0]!r}"


@pytest.mark.parametrize("kind,M,K,rank", [("b3", 1, 768, 8), ("b3", 2, 1536, 40), ("b3", 3, 768, 8), ("short", 8, 64, 8),
                                           ("direct", 24, 64, 40), ("direct", 6, 4104, 8), ("queue", 5, 64, 40)])
def test_gate_of_every_fp16(kind, M, K, rank):
    bits = np.arange(65536, dtype=np.uint16).view(np.float16)
    alphas = bits[np.isfinite(bits)]
    for part in np.split(alphas, 2 if kind == "short" else 1):       # (32768 rows are the most that one launch takes)
        _check_gates(kind, M, K, rank, part)


def _check_gates(kind, M, K, rank, alphas):
    N = len(alphas)
    ws = hb.Workspace(M, K, N, rank)
    L = _layer(K, N, rank, 32.0, torch.from_numpy(alphas.copy()).cuda(), ws, b3=kind == "b3")
    x = _tokens(M, K, 1024.0)
    if kind == "queue":                      # five phases, each with tokens of its own
        ys = [torch.empty((M, N), dtype=torch.float16, device="cuda") for _ in range(5)]
        xs = [x.clone() for _ in range(5)]
        layers = [hb.Layer(L.packed, L.s_w, N, K, L.A, L.B, L.alpha, src_slot=i, dst_slot=5 + i) for i in range(5)]
        before = int(ws.buf[:64].view(torch.int32)[8])
        hb.hgf_stack_forward(hb.Stack(layers, xs + ys, M), ws)
        assert int(ws.buf[:64].view(torch.int32)[8]) == before + 1
    else:
        ys = [(hb.hgf_linear_forward_b3 if kind == "b3" else hb.hgf_linear_forward)(x, L, ws)]
    exact = np.broadcast_to(np.tanh(alphas.astype(np.float64)) * 32768, (M, N))
    for y in ys:
        _assert_rounded(y.cpu().numpy(), exact, 2.0 ** -21)


@pytest.mark.parametrize("kind,K,rank", [("short", 64, 8), ("direct", 64, 40)])
def test_silu_of_a_gated_pair(kind, K, rank):
    M, N = 24, 8192
    rng = np.random.default_rng(7)
    half = lambda v: v.astype(np.float16)
    h, bg, bu = half(32 + rng.integers(0, 32, M)), half(-rng.uniform(0.06, 0.28, N)), half(rng.uniform(4, 16, N))
    one = torch.full((N,), 20.0, dtype=torch.float16, device="cuda")     # its gate is 1 in fp32
    ws = hb.Workspace(M, K, N, rank)
    g, u = (_layer(K, N, rank, torch.from_numpy(b).cuda(), one, ws) for b in (bg, bu))
    z = hb.hgf_swiglu_forward(_tokens(M, K, torch.from_numpy(h).cuda()), g, u, ws).cpu().numpy()
    yg, yu = (h.astype(np.float64)[:, None] * b.astype(np.float64) for b in (bg, bu))    # (exact in fp32)
    _assert_rounded(z, yg / (1 + np.exp(-yg)) * yu, 2.4e-7)
