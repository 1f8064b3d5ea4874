"""GPU parity where the direct path and the prefill path can go wrong: edges of the direct kernel's
32 x 32 tiles and of its token groups, the shapes its dispatch chooses between, d_in cut into slices for
A x, rows that are not 16-byte aligned -- and the prefill kernel at sizes the direct path leaves to it.
Accumulators bit for bit, outputs within 2e-3 + 1e-2 |y| (fp16 rounding of h and y)."""
import numpy as np
import pytest
import torch

from paper_2602_05269_amd import binding as hb
from paper_2602_05269_amd import synth
from parity import GpuLayer, assert_close_fp16, dev, path_taken
from test_gpu_layernorm import LnLayer
from test_gpu_swiglu import _check_pair

pytestmark = pytest.mark.gpu


def _one(M, K, N, r, act="student_t3", path="direct"):
    c = synth.make_custom(5000 + M + K + N + r, M, K, N, max(r, 1), act=act, lora_std=0.05)
    g = GpuLayer(c, hb.Workspace(M, K, N, max(r, 1)), rank0=r == 0)
    with path_taken(path):
        y, acc = g.forward(c["x"])
    ref = g.oracle(c["x"], dense=True)
    assert np.array_equal(acc, ref["acc"]), "int32 accumulators differ from the oracle"
    assert_close_fp16(y, ref["y"])


@pytest.mark.parametrize("M,K,N,r", [
    # token groups: full, one over, two full, ragged third; row-blocks: one, ragged, odd number
    (31, 128, 32, 16), (32, 129, 33, 8), (33, 255, 95, 24), (64, 384, 160, 0), (65, 130, 1, 128), (97, 640, 225, 40),
    # eight wavefronts along d_in; more k-tiles than wavefronts x tiles in flight
    (5, 4104, 64, 16), (8, 8320, 40, 128), (40, 11000, 96, 100),
    # two row-blocks per workgroup: 280 .. 640 tiles and more, an odd number of row-blocks
    (70, 520, 3000, 20), (130, 264, 4128, 16), (200, 2056, 2999, 64),
    # slices of d_in for A x: 2, 3, 5 and 9 of them, the last one ragged; rows at odd addresses
    (7, 2049, 64, 16), (6, 4097, 33, 32), (20, 10001, 40, 128), (5, 16500, 32, 8), (9, 1365, 512, 16), (50, 4095, 70, 15),
    # two token tiles per workgroup of A x (more than 512 workgroups otherwise), each quantiser width
    (1050, 130, 32, 128), (1040, 1416, 40, 128), (1040, 2056, 32, 64), (530, 4104, 33, 128),
    # a row longer than what the quantiser keeps in registers
    (6, 16640, 40, 24), (5, 33001, 32, 8),
])
def test_direct_path_edges(M, K, N, r):
    _one(M, K, N, r)


@pytest.mark.parametrize("M,K,N,r", [
    # one token group and many row-blocks: one tile in flight up to 1300 row-blocks of 8 k-tiles, up to 800 of 24,
    # and of longer rows with read-once requests; two row-blocks per workgroup up to 1050 and beyond (short and
    # long rows), an odd number of them, the last one ragged
    (9, 520, 9000, 16), (32, 1024, 41569, 8), (5, 3072, 8225, 24), (17, 3080, 16417, 8), (31, 1100, 25665, 40),
    (6, 500, 41633, 16), (8, 1100, 33633, 0),
])
def test_direct_path_many_row_blocks(M, K, N, r):
    _one(M, K, N, r)


@pytest.mark.parametrize("M,K,N,r", [
    (600, 1365, 4096, 32), (900, 256, 3000, 16), (1000, 4104, 2048, 8), (1000, 8200, 2400, 16), (1000, 16392, 2400, 8),
    (1000, 512, 2100, 0), (1040, 2056, 32, 120),
    # odd rows: ranks padded to 64 and 128 columns, rows read once per pass
    (1000, 1365, 2100, 40), (700, 1001, 4100, 100), (700, 16401, 3600, 8),
])
def test_prefill_path(M, K, N, r):
    """Sizes beyond the direct path: the three register depths of the prefill quantiser, ragged row and
    token tiles, odd rows, no correction path."""
    _one(M, K, N, r, act="student_t4", path="prefill")


@pytest.mark.parametrize("M,K,N,r,path", [
    # the line between the paths, a row-block on either side of it: up to 2048 columns, up to 6144, beyond
    (200, 512, 7520, 16, "direct"), (200, 512, 7553, 16, "prefill"), (640, 2048, 2208, 64, "direct"), (640, 2048, 2209, 64, "prefill"),
    # no ranks: odd rows of up to 512 columns, longer ones
    (320, 137, 3648, 0, "direct"), (320, 137, 3649, 0, "prefill"), (320, 511, 3649, 0, "prefill"), (320, 513, 3649, 0, "direct"),
    (640, 2049, 2432, 48, "direct"), (640, 2049, 2433, 48, "prefill"), (640, 6152, 3712, 0, "direct"), (640, 6152, 3713, 0, "prefill"),
    # many tokens, few rows: 2000 x (1/2 + 1/4) - 512/4 = 1372 and 6 tiles of 63 rows
    (2000, 264, 192, 8, "direct"), (2000, 264, 193, 8, "prefill"), (1300, 2056, 512, 8, "direct"), (1300, 2056, 1248, 8, "prefill"),
])
def test_line_between_the_paths(M, K, N, r, path):
    _one(M, K, N, r, path=path)


@pytest.mark.parametrize("M,K,N,path", [
    # up to 512 columns, up to 2048, beyond
    (320, 512, 7168, "direct"), (320, 512, 7169, "prefill"), (320, 520, 6528, "direct"), (320, 520, 6529, "prefill"),
    (320, 2056, 6784, "direct"), (320, 2056, 6817, "prefill"),
    # prefill of more than 4096 columns: prepared in one launch, in two
    (900, 4504, 2400, "prefill"), (1000, 4496, 2200, "prefill"),
    # ... and the line where it is two
    (1000, 4992, 1088, "direct"), (1000, 4992, 1089, "prefill"), (998, 4992, 1089, "direct"),
])
def test_line_between_the_paths_behind_a_layernorm(M, K, N, path):
    c = synth.make_custom(8950 + M + K + N, M, K, N, 16, act="student_t3", lora_std=0.05)
    g = LnLayer(c, hb.Workspace(M, K, N, 16), seed=M + K)
    with path_taken(path):
        y, acc = g.forward(c["x"])
    ref = g.oracle(c["x"], dense=True)
    assert np.array_equal(acc, ref["acc"]), "int32 accumulators differ from the oracle"
    assert_close_fp16(y, ref["y"])


@pytest.mark.parametrize("M,K,N,path", [
    # up to 512 columns, where a workgroup per token prepares, and beyond, where the prologue does
    (320, 512, 6208, "direct"), (320, 512, 6209, "prefill"), (320, 520, 6209, "direct"), (320, 137, 3648, "direct"),
    (320, 137, 3649, "prefill"), (320, 511, 3649, "prefill"), (600, 1025, 4100, "prefill"),
])
def test_line_between_the_paths_behind_a_layernorm_without_ranks(M, K, N, path):
    c = synth.make_custom(8990 + M + K + N, M, K, N, 1, act="student_t3", lora_std=0.05)
    g = LnLayer(c, hb.Workspace(M, K, N, 1), seed=M + K, rank0=True)
    with path_taken(path):
        y, acc = g.forward(c["x"])
    ref = g.oracle(c["x"], dense=True)
    assert np.array_equal(acc, ref["acc"]), "int32 accumulators differ from the oracle"
    assert_close_fp16(y, ref["y"])


@pytest.mark.parametrize("M,K,N,r,ln,path", [
    (9, 130, 40, 1, False, "direct"), (50, 2500, 40, 5, False, "direct"), (600, 1365, 4096, 1, False, "prefill"),
    (600, 1360, 4096, 17, False, "prefill"), (900, 1360, 4096, 16, True, "prefill"), (900, 1365, 4096, 3, True, "prefill"),
])
def test_infinite_activation_stays_out_of_padded_ranks(M, K, N, r, ln, path):
    """One token holds +inf where every row of A is positive, so SiLU(A x) is +inf for every rank, and with
    B and the gate positive the correction is +inf; a rank that pads the tile (a zero row of A: 0 * inf is
    NaN) must not reach it.  The integer sum of that column's code (-127: inf * 0 is NaN, which the clip
    turns into the lower bound) gives +inf where T is -1; behind a LayerNorm every code of the token is -127."""
    c = synth.make_custom(5900 + M + K + r, M, K, N, r, act="normal", lora_std=0.05)
    c["A"], c["B"], c["alpha"] = np.abs(c["A"]) + np.float16(0.01), np.abs(c["B"]) + np.float16(0.01), np.abs(c["alpha"]) + np.float16(0.1)
    x = c["x"].copy()
    m, k = M // 2, K // 3
    x[m, k] = np.inf
    ws = hb.Workspace(M, K, N, r)
    g = LnLayer(c, ws, seed=1) if ln else GpuLayer(c, ws)
    with path_taken(path):
        y, acc = g.forward(x)
    if ln:
        # amax of an all-NaN row is the floor: a finite term beside the infinite correction
        assert (y[m] == np.inf).all()
    else:
        assert np.array_equal(acc[m], -127 * g.T_ref[:, k].astype(np.int32))
        assert (g.T_ref[:, k] == -1).any() and (y[m, g.T_ref[:, k] == -1] == np.inf).all()
    others = np.arange(M) != m
    assert_close_fp16(y[others], g.oracle(x[others], dense=True)["y"])


@pytest.mark.parametrize("M", [150, 2000])
def test_groups_of_mixed_layers(M):
    """Four layers of mixed ranks and ragged d_out read one slot, on the direct path (150 tokens) and on
    the prefill path (2000; rank 64 pads to another width and takes a launch of its own): against the
    oracle."""
    K = 384
    shapes = [(300, 16), (256, 24), (40, 32), (128, 64)]
    cases, layers, slots = [], [], [None] * (len(shapes) + 1)
    ws = hb.Workspace(M, K, 384, 64)
    for i, (N, r) in enumerate(shapes):
        c = synth.make_custom(8700 + i, M, K, N, r, act="student_t4", lora_std=0.05, w_std=0.05)
        if i == 0:
            x = c["x"]
            slots[0] = dev(x)
        g = GpuLayer(c, ws)
        g.layer.c.src_slot, g.layer.c.dst_slot = 0, i + 1
        cases.append(g)
        layers.append(g.layer)
        slots[i + 1] = torch.zeros((M, N), dtype=torch.float16, device="cuda")
    with path_taken("direct" if M == 150 else "prefill"):
        hb.hgf_stack_forward(hb.Stack(layers, slots, M), ws)
    torch.cuda.synchronize()
    for i, g in enumerate(cases):
        assert_close_fp16(slots[i + 1].cpu().numpy(), g.oracle(x, dense=True)["y"], f"layer {i}")


@pytest.mark.parametrize("ln", [False, True])
def test_group_with_room_for_some_slices(ln):
    """Three layers of 9000 columns at 700 tokens: A x would be cut into five slices, the workspace holds
    three; behind LayerNorms, where it also holds two further quantisations, 190 tokens leave room for two."""
    M, K, r = (190, 9000, 128) if ln else (700, 9000, 32)
    ws = hb.Workspace(M, K, 40, r)
    layers, cases, slots = [], [], [None] * 4
    for i, N in enumerate((40, 33, 8)):
        c = synth.make_custom(8900 + i, M, K, N, r, act="student_t4", lora_std=0.01, w_std=0.05)
        if i == 0:
            x = c["x"]
            slots[0] = dev(x)
        g = LnLayer(c, ws, seed=i) if ln else GpuLayer(c, ws)
        g.layer.c.src_slot, g.layer.c.dst_slot = 0, i + 1
        slots[i + 1] = torch.zeros((M, N), dtype=torch.float16, device="cuda")
        cases.append(g)
        layers.append(g.layer)
    with path_taken("direct"):
        hb.hgf_stack_forward(hb.Stack(layers, slots, M), ws)
    torch.cuda.synchronize()
    for i, g in enumerate(cases):
        assert_close_fp16(slots[i + 1].cpu().numpy(), g.oracle(x, dense=True)["y"], f"layer {i}")


def test_more_tokens_than_one_launch_prepares():
    """Four layers of odd rows and 65 to 128 ranks read 7.6 million tokens: their preparation is more threads
    than a launch may have, so it goes out layer by layer.  A few tokens from either end against the oracle."""
    M, K, N = 7_600_000, 33, 8
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    x = torch.randn((M, K), generator=gen, device="cuda", dtype=torch.float16)
    ws = hb.Workspace(M, K, N, 128)
    layers, cases, slots = [], [], [x]
    for i, r in enumerate((128, 65, 100, 0)):
        c = synth.make_custom(8990 + i, 1, K, N, max(r, 1), act="normal", lora_std=0.05, w_std=0.05)
        g = GpuLayer(c, ws, rank0=r == 0)
        g.layer.c.src_slot, g.layer.c.dst_slot = 0, i + 1
        slots.append(torch.zeros((M, N), dtype=torch.float16, device="cuda"))
        cases.append(g)
        layers.append(g.layer)
    hb.hgf_stack_forward(hb.Stack(layers, slots, M), ws)
    torch.cuda.synchronize()
    some = torch.cat([torch.arange(40), torch.arange(M // 2, M // 2 + 40), torch.arange(M - 40, M)])
    xs = x[some.cuda()].cpu().numpy()
    for i, g in enumerate(cases):
        assert_close_fp16(slots[i + 1][some.cuda()].cpu().numpy(), g.oracle(xs)["y"], f"layer {i}")


@pytest.mark.parametrize("M,K,N,rg,ru,path", [
    # eight and four wavefronts, ragged rows of the last row-block, sliced A x, one rank zero, many row-blocks
    (33, 130, 65, 24, 8, "direct"), (40, 2500, 300, 16, 40, "direct"), (50, 2500, 300, 16, 24, "direct"),
    (64, 300, 4500, 8, 0, "direct"), (10, 9000, 70, 0, 128, "direct"), (330, 384, 2100, 0, 0, "direct"),
    (3, 1100, 8225, 16, 24, "direct"), (32, 2056, 8200, 0, 40, "direct"),
    (400, 1365, 2050, 32, 0, "prefill"), (450, 384, 2100, 0, 0, "prefill"), (400, 4104, 2000, 16, 24, "prefill"),
    # a row-block on either side of the line: up to 2048 columns, up to 6144, beyond
    (320, 1024, 2528, 16, 16, "direct"), (320, 1024, 2529, 16, 16, "prefill"), (320, 2056, 2272, 32, 32, "direct"),
    (320, 2056, 2273, 32, 32, "prefill"), (320, 6152, 4032, 16, 0, "direct"), (320, 6152, 4033, 16, 0, "prefill"),
])
def test_pair_paths(M, K, N, rg, ru, path):
    ws = hb.Workspace(M, K, N, max(rg, ru, 1))
    # A x of order one: the fp16 rounding of h moves y_up by up to 2^-11 sum_j |B h|, and z by SiLU(y_gate)
    # times that; with std 0.05 at d_in = 9000, |h| ~ 5, 128 ranks and SiLU(y_gate) ~ 5 it is 8e-3, beyond
    # the 2e-3 that are allowed where z itself is near zero (seen: 1 of 700 elements)
    std = min(0.05, 1.0 / np.sqrt(K))
    cg = synth.make_custom(8400 + M + K + N + rg, M, K, N, max(rg, 1), act="student_t3", lora_std=std)
    cu = synth.make_custom(8450 + M + K + N + ru, M, K, N, max(ru, 1), act="student_t3", lora_std=std)
    gate, up = GpuLayer(cg, ws, rank0=rg == 0), GpuLayer(cu, ws, rank0=ru == 0)
    with path_taken(path):
        _check_pair(gate, up, cg["x"], ws, dense=True)


@pytest.mark.parametrize("M,K,N,r", [
    # direct: a wavefront, 128, 256 and 512 threads per token, rows read once per pass, odd rows
    (70, 96, 40, 8), (9, 1030, 64, 16), (6, 2048, 33, 24), (6, 4097, 33, 32), (5, 9001, 70, 8), (6, 16640, 40, 24), (5, 33001, 32, 0),
    # prefill: prepared in one launch, in two
    (900, 1365, 4096, 32), (1900, 512, 2100, 0), (1000, 2048, 2500, 40), (1100, 8192, 1800, 16),
])
def test_layernorm_paths(M, K, N, r):
    c = synth.make_custom(8600 + M + K + N + r, M, K, N, max(r, 1), act="student_t3", lora_std=0.05)
    g = LnLayer(c, hb.Workspace(M, K, N, max(r, 1)), seed=M + K, rank0=r == 0, with_beta=M % 2 == 1)
    y, acc = g.forward(c["x"])
    ref = g.oracle(c["x"], dense=True)
    assert np.array_equal(acc, ref["acc"]), "int32 accumulators differ from the oracle"
    assert_close_fp16(y, ref["y"])


@pytest.mark.parametrize("M,K,r", [(3, 100, 8), (40, 1365, 16), (500, 512, 32), (33, 3000, 24), (6, 512, 0)])
@pytest.mark.parametrize("shared", [False, True])
def test_layernorm_layers_of_one_input(M, K, r, shared):
    """Three layers with LayerNorms of their own read one slot (quantised together where the workspace
    has room: not with rank 0); with shared memory the first one's output slot is the input itself, which
    the two others then read."""
    ws = hb.Workspace(M, K, max(K, 520), r)
    widths = (K if shared else 520, 96, 33)
    slots, cases, layers = [None] * 4, [], []
    for i, N in enumerate(widths):
        c = synth.make_custom(8800 + M + 7 * i, M, K, N, max(r, 1), act="student_t4", lora_std=0.02, w_std=0.05)
        if i == 0:
            x = c["x"]
            slots[0] = dev(x)
        g = LnLayer(c, ws, seed=i + K, rank0=r == 0, with_beta=i != 1)
        g.layer.c.src_slot, g.layer.c.dst_slot, g.layer.c.ln_eps = 0, i + 1, 1e-5
        slots[i + 1] = slots[0] if shared and i == 0 else torch.zeros((M, N), dtype=torch.float16, device="cuda")
        cases.append(g)
        layers.append(g.layer)
    hb.hgf_stack_forward(hb.Stack(layers, slots, M), ws)
    torch.cuda.synchronize()
    out = [s.cpu().numpy() for s in slots]
    assert_close_fp16(out[1], cases[0].oracle(x, dense=True)["y"], "layer 0")
    for i in (1, 2):
        assert_close_fp16(out[i + 1], cases[i].oracle(out[0], dense=True)["y"], f"layer {i}")
