"""GPU parity of the launch for short rows (every workgroup prepares its own tokens): each of its shapes
(tokens per workgroup, wavefronts per row-block, pieces per thread), ragged tokens, rows, ranks and columns,
with and without LayerNorm, single, grouped and as a SwiGLU pair.  Accumulators bit for bit, outputs within
2e-3 + 1e-2 |y| (fp16 rounding of h and y)."""
import ctypes

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


class _KernelNode(ctypes.Structure):           # hipKernelNodeParams
    _fields_ = [("block", ctypes.c_uint * 3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p),
                ("grid", ctypes.c_uint * 3), ("params", ctypes.c_void_p), ("lds", ctypes.c_uint)]


def _launches(call):
    """(threads, workgroups) of every kernel that `call` launches, from a capture of it."""
    hip = ctypes.CDLL(next(l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l))
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        call()
    raw = ctypes.c_void_p(graph.raw_cuda_graph())
    n = ctypes.c_size_t(0)
    assert hip.hipGraphGetNodes(raw, None, ctypes.byref(n)) == 0
    nodes = (ctypes.c_void_p * n.value)()
    assert hip.hipGraphGetNodes(raw, nodes, ctypes.byref(n)) == 0
    out = []
    for node in nodes:
        k = _KernelNode()
        assert hip.hipGraphKernelNodeGetParams(ctypes.c_void_p(node), ctypes.byref(k)) == 0
        out.append((k.block[0] * k.block[1] * k.block[2], k.grid[0] * k.grid[1] * k.grid[2]))
    return out


@pytest.mark.parametrize("bad", [None, np.inf, np.nan])
@pytest.mark.parametrize("kind,M,K,N,r,tokens,ks", [
    # tokens of a workgroup and wavefronts per row-block that the rule chooses; with the columns they give the pieces
    # per thread (1, 2 or 4) and, beyond 512, two steps of A x
    ("plain", 8, 512, 33, 16, 8, 8), ("plain", 7, 1024, 95, 32, 8, 8), ("plain", 9, 2048, 64, 16, 8, 8), ("plain", 48, 512, 1400, 24, 16, 8),
    ("plain", 40, 256, 2000, 16, 16, 8), ("plain", 100, 512, 1333, 16, 16, 4), ("plain", 100, 256, 1333, 16, 16, 4),
    ("plain", 64, 1000, 3200, 16, 16, 4), ("plain", 250, 512, 1060, 32, 32, 4), ("plain", 255, 512, 2100, 8, 32, 2),
    ("plain", 255, 256, 2100, 8, 32, 2), ("plain", 255, 128, 2100, 8, 32, 2),
    ("plain", 13, 65, 100, 17, 8, 8), ("plain", 50, 511, 1300, 16, 16, 8), ("plain", 300, 333, 640, 3, 16, 4), ("plain", 300, 201, 640, 3, 16, 4),
    ("plain", 300, 333, 1280, 3, 32, 4), ("plain", 300, 511, 2400, 3, 32, 2), ("plain", 300, 250, 2400, 3, 32, 2),
    ("plain", 300, 100, 2400, 3, 32, 2),
    ("ln", 40, 512, 1500, 16, 8, 8), ("ln", 120, 512, 1061, 16, 8, 4), ("ln", 100, 1024, 960, 16, 8, 4), ("ln", 24, 1024, 400, 16, 8, 8),
    ("ln", 300, 512, 700, 16, 16, 4), ("ln", 300, 512, 1280, 16, 16, 2), ("ln", 500, 512, 1500, 16, 16, 1), ("ln", 300, 200, 1280, 16, 16, 2),
    ("ln", 500, 128, 1500, 16, 16, 1), ("ln", 24, 255, 300, 16, 8, 8), ("ln", 120, 251, 1000, 5, 8, 4), ("ln", 300, 201, 1280, 16, 16, 2), ("ln", 500, 250, 1500, 5, 16, 1),
    ("pair", 24, 512, 1365, 16, 8, 8), ("pair", 60, 504, 1400, 16, 16, 8), ("pair", 130, 256, 1100, 16, 16, 4), ("pair", 400, 128, 1000, 8, 32, 4),
    ("pair", 400, 120, 1700, 8, 32, 2), ("pair", 33, 77, 320, 5, 8, 8), ("pair", 24, 1000, 900, 16, 8, 8), ("pair", 100, 1000, 640, 16, 16, 8),
    ("pair", 100, 1000, 1600, 16, 16, 4), ("pair", 60, 500, 1400, 16, 16, 8), ("pair", 130, 333, 1100, 5, 16, 4), ("pair", 130, 336, 1100, 8, 16, 4),
    ("pair", 200, 504, 1300, 8, 32, 4), ("pair", 200, 501, 1300, 5, 32, 4), ("pair", 130, 201, 1100, 5, 16, 4), ("pair", 400, 248, 1700, 8, 32, 2),
    ("pair", 400, 201, 1700, 5, 32, 2), ("pair", 400, 101, 1700, 5, 32, 2),
])
def test_shape_and_bits_of_two_launches(kind, M, K, N, r, tokens, ks, bad):
    """The rule's choice, seen in the captured launch, and the same bits as the two launches of level 0, also for tokens
    that hold an infinity or what is not a number."""
    ws = hb.Workspace(M, K, N, r)
    cases = [synth.make_custom(6700 + i, M, K, N, r, act="student_t4", lora_std=0.05, w_std=0.05) for i in range(2 if kind == "pair" else 1)]
    gs = [LnLayer(c, ws, seed=M + K) if kind == "ln" else GpuLayer(c, ws) for c in cases]
    x = cases[0]["x"].copy()
    if bad is not None:
        x[M // 2, K // 3] = bad
        x[0, K - 1] = -bad
    xd = dev(x)
    out = torch.empty((M, N), dtype=torch.float16, device="cuda")
    accs = [torch.empty((M, N), dtype=torch.int32, device="cuda") for _ in gs]

    def call():
        if kind == "pair":
            hb.hgf_swiglu_forward(xd, gs[0].layer, gs[1].layer, ws, z=out, acc_debug_gate=accs[0], acc_debug_up=accs[1])
        else:
            hb.hgf_linear_forward(xd, gs[0].layer, ws, y=out, acc_debug=accs[0])

    got = []
    for level in (2, 0):
        hb.hgf_set_single_launch(level)
        try:
            call()
            got.append([out.cpu().numpy().copy()] + [a.cpu().numpy().copy() for a in accs])
            if bad is None:
                seen = _launches(call)
                if level == 2:
                    assert seen == [(512, -(-M // tokens) * -(-(-(-N // 32)) * ks // 8))], seen
                else:
                    assert len(seen) == 2, seen
        finally:
            hb.hgf_set_single_launch(2)
    one, two = got
    assert np.array_equal(np.isnan(one[0]), np.isnan(two[0]))
    fine = ~np.isnan(one[0])
    assert np.array_equal(one[0][fine].view(np.uint16), two[0][fine].view(np.uint16))
    for a, b in zip(one[1:], two[1:]):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("kind,M,K,N,r,one", [
    # behind LayerNorms: 15 token groups of 3 x 5 workgroups, of 3 x 6 (more than 256), which a sum over all rows hides
    ("ln3", 114, 688, 320, 16, True), ("ln3", 114, 688, 336, 16, False),
    # several row-blocks whose rows of B are no whole pieces; few tokens behind a LayerNorm; pairs; eight row-blocks
    ("plain", 64, 1000, 3200, 24, True), ("plain", 64, 1000, 3200, 17, False), ("plain", 32, 536, 2940, 17, True),
    ("ln", 250, 512, 2300, 16, False), ("ln", 256, 512, 2300, 16, True), ("ln", 250, 256, 2300, 16, True),
    ("pair", 400, 264, 1700, 8, False), ("plain", 500, 264, 2050, 16, False),
])
def test_edges_of_the_rule(kind, M, K, N, r, one):
    ws = hb.Workspace(M, K, N, r)
    n = {"ln3": 3, "pair": 2}.get(kind, 1)
    cases = [synth.make_custom(6900 + i, M, K, N, r, act="student_t4", lora_std=0.05, w_std=0.05) for i in range(n)]
    gs = [LnLayer(c, ws, seed=i) if kind in ("ln", "ln3") else GpuLayer(c, ws) for i, c in enumerate(cases)]
    x, ys = dev(cases[0]["x"]), [torch.empty((M, N), dtype=torch.float16, device="cuda") for _ in gs]
    for i, g in enumerate(gs):
        g.layer.c.src_slot, g.layer.c.dst_slot = 0, i + 1
    st = hb.Stack([g.layer for g in gs], [x] + ys, M)

    def call():
        if kind == "pair":
            hb.hgf_swiglu_forward(x, gs[0].layer, gs[1].layer, ws, z=ys[0])
        else:
            hb.hgf_stack_forward(st, ws)

    call()
    assert (len(_launches(call)) == 1) == one
