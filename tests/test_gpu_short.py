"""GPU parity of the launch for short rows (every workgroup prepares its own tokens): each of its shapes
(tokens per workgroup, wavefronts per row-block, pieces per thread), ragged tokens, rows, ranks and columns,
with and without LayerNorm, single, grouped and as a SwiGLU pair.  Accumulators bit for bit, outputs within
2e-3 + 1e-2 |y| (fp16 rounding of h and y)."""
import numpy as np
import pytest
import torch

from paper_2602_05269_amd import binding as hb
from paper_2602_05269_amd import synth
from parity import GpuLayer, assert_close_fp16, dev
from test_gpu_layernorm import LnLayer
from test_gpu_swiglu import _check_pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,N,r", [
    # 8 tokens and one row-block per workgroup: one, two and four pieces of 8 columns per thread
    (5, 8, 1, 1), (8, 512, 33, 16), (7, 1024, 95, 32), (9, 2048, 64, 16), (31, 2040, 31, 0),
    # 16 tokens; two row-blocks; 32 tokens with two, four and eight row-blocks per workgroup
    (48, 512, 1400, 24), (100, 512, 1333, 16), (250, 512, 1060, 32), (255, 256, 2100, 8), (500, 264, 2050, 16),
    # columns at odd addresses
    (6, 1, 40, 3), (13, 65, 100, 17), (33, 333, 700, 32), (300, 511, 95, 16), (40, 131, 2000, 5),
    # more columns than one step of A x, k-tiles that do not divide over the wavefronts
    (24, 1160, 160, 16), (64, 640, 512, 20),
])
def test_short_rows(M, K, N, r):
    c = synth.make_custom(6000 + M + K + N + r, M, K, N, max(r, 1), act="student_t3", lora_std=0.05)
    g = GpuLayer(c, hb.Workspace(M, K, N, max(r, 1)), rank0=r == 0)
    y, acc = g.forward(c["x"])
    ref = g.oracle(c["x"], dense=True)
    assert np.array_equal(acc, ref["acc"]), "int32 accumulators differ from the oracle"
    assert_close_fp16(y, ref["y"])


@pytest.mark.parametrize("M,K,N", [
    (1, 512, 40), (8, 1024, 33), (40, 512, 1500), (120, 512, 1061), (300, 512, 700), (500, 512, 1500), (24, 255, 300), (7, 2, 5),
])
def test_short_rows_behind_a_layernorm(M, K, N):
    c = synth.make_custom(6200 + M + K + N, M, K, N, 16, act="student_t3", lora_std=0.05)
    g = LnLayer(c, hb.Workspace(M, K, N, 16), seed=M + K)
    y, acc = g.forward(c["x"])
    ref = g.oracle(c["x"], dense=True)
    assert np.array_equal(acc, ref["acc"]), "int32 accumulators differ from the oracle"
    assert_close_fp16(y, ref["y"])


@pytest.mark.parametrize("M,K,N,r,r2", [(1, 512, 65, 16, 16), (24, 512, 1365, 16, 8), (60, 500, 1400, 16, 16), (130, 256, 1100, 0, 16),
                                        (400, 128, 1000, 16, 0), (33, 77, 320, 5, 16)])
def test_short_rows_as_a_pair(M, K, N, r, r2):
    cg = synth.make_custom(6400 + M + K, M, K, N, max(r, 1), act="student_t3", lora_std=0.05)
    cu = synth.make_custom(6500 + M + K, M, K, N, max(r2, 1), act="student_t3", lora_std=0.05)
    ws = hb.Workspace(M, K, N, 16)
    _check_pair(GpuLayer(cg, ws, rank0=r == 0), GpuLayer(cu, ws, rank0=r2 == 0), cg["x"], ws)


@pytest.mark.parametrize("M", [8, 150, 400])
@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_short_rows_give_the_bits_of_two_launches(M, bad):
    """The same layers in a group with one of many ranks, which takes the direct path's two launches: equal
    bits, also for tokens that hold an infinity or what is not a number."""
    K, N = 384, 200
    ws = hb.Workspace(M, K, N, 64)
    cases = [synth.make_custom(6600 + i, M, K, N, max(r, 1), act="student_t4", lora_std=0.05, w_std=0.05) for i, r in enumerate((64, 24, 1))]
    x = cases[0]["x"].copy()
    x[M // 2, 5] = bad
    x[0, K - 1] = bad
    gs = [GpuLayer(c, ws, rank0=i == 2) for i, c in enumerate(cases)]
    slots = [dev(x)] + [torch.zeros((M, N), dtype=torch.float16, device="cuda") for _ in gs]
    for i, g in enumerate(gs):
        g.layer.c.src_slot, g.layer.c.dst_slot = 0, i + 1
    hb.hgf_stack_forward(hb.Stack([g.layer for g in gs], slots, M), ws)
    for i, g in enumerate(gs[1:]):
        y, _ = g.forward(x)
        two = slots[i + 2].cpu().numpy()
        assert np.array_equal(np.isnan(y), np.isnan(two))
        assert np.array_equal(y[~np.isnan(y)].view(np.uint16), two[~np.isnan(y)].view(np.uint16))
