"""GPU parity: the HIP path (through the C ABI) against the CPU oracle, element by element
on the same seeded inputs.  Integers (codes, x_q, rowsum, int32 accumulators) and the fp32
scales bit-exact; fp16 outputs within 2e-3 + 1e-2 |y|."""
import numpy as np
import pytest
import torch

from oracle import hgf_oracle as orc
from paper_2602_05269_amd import binding as hb
from paper_2602_05269_amd import synth
from parity import GpuLayer, assert_close_fp16, dev, path_taken

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ws():
    return hb.Workspace(2048, 11008, 11008, 128)


# ------------------------------------------------------------------ quantiser

@pytest.mark.parametrize("M,K,kind", [(1, 1, "normal"), (3, 63, "normal"), (8, 256, "normal"), (5, 1365, "student_t3"),
                                      (16, 2048, "outlier"), (7, 11008, "student_t3"), (300, 3072, "student_t4")])
def test_quantize_activations_bit_exact(M, K, kind):
    x = synth.draw_activations(kind, np.random.default_rng([M, K]), M, K)
    if M >= 3:
        x[1] = 0                                       # an all-zero token
        x[2, K // 2] = np.float16(60000.0)             # a huge outlier
    xq, s_x, rowsum = hb.hgf_quantize_activations(dev(x))
    torch.cuda.synchronize()
    xq_ref, s_ref, rs_ref = orc.quantize_act(x)
    xq = xq.cpu().numpy()
    assert np.array_equal(xq[:, :K], xq_ref)
    assert not xq[:, K:].any()                         # padding columns are zero
    assert np.array_equal(s_x.cpu().numpy().view(np.uint32), s_ref.view(np.uint32))
    assert np.array_equal(rowsum.cpu().numpy(), rs_ref)


# ------------------------------------------------------------------ weights

@pytest.mark.parametrize("N,K", [(1, 1), (3, 63), (64, 64), (65, 65), (100, 1365), (256, 256), (2048, 512)])
def test_pack_unpack_matches_oracle_ternariser(N, K, ws):
    c = synth.make_custom(N * 7 + K, 1, K, N, 8)
    g = GpuLayer(c, ws)
    g.check_weights()


@pytest.mark.parametrize("N,K", [(1, 1), (2, 3), (35, 4), (3, 5), (34, 6), (5, 7), (31, 127), (33, 129), (32, 130), (65, 259), (3, 1365)])
def test_pack_edges_of_tiles_and_odd_addresses(N, K, ws):
    # edges of the 32 x 128 tiles, one to three columns past the last whole 16 bytes, and latents that
    # start at any multiple of four bytes; padding rows and columns hold code 1 (bytes of 0x55)
    W = np.random.default_rng(N * 7919 + K).standard_normal((N, K)).astype(np.float32)
    T, s_w = orc.ternarize(W)
    for shift in range(4):
        flat = torch.zeros(N * K + 4, dtype=torch.float32, device="cuda")
        flat[shift:shift + N * K] = dev(W).flatten()
        packed, s = hb.hgf_quantize_pack_weights(flat[shift:shift + N * K].view(N, K), ws)
        assert s.item() == float(s_w)
        assert np.array_equal(hb.hgf_unpack_weights(packed, N, K).cpu().numpy(), T)
        padded = hb.hgf_unpack_weights(packed, -(-N // 32) * 32, -(-K // 128) * 128).cpu().numpy()
        assert not padded[N:].any() and not padded[:, K:].any()


def test_pack_constructed_ties_and_zero_matrix(ws):
    W = np.array([[0.5, -0.5, 1.5, -1.5], [0.25, -0.25, 1.75, -1.75]], dtype=np.float32)
    packed, s_w = hb.hgf_quantize_pack_weights(dev(W), ws)
    T = hb.hgf_unpack_weights(packed, 2, 4).cpu().numpy()
    assert s_w.item() == 1.0 and T.tolist() == [[0, 0, 1, -1], [0, 0, 1, -1]]
    packed, s_w = hb.hgf_quantize_pack_weights(dev(np.zeros((5, 70), dtype=np.float32)), ws)
    assert s_w.cpu().numpy()[0] == np.float32(1e-5)
    assert not hb.hgf_unpack_weights(packed, 5, 70).cpu().numpy().any()
    # padding codes decode to zero: every 2-bit field of the buffer is 0, 1 or 2, padding is 1
    raw = packed.cpu().numpy()
    fields = np.stack([(raw >> s) & 3 for s in (0, 2, 4, 6)])
    assert (fields == 1).all()


# ------------------------------------------------------------------ one layer

def test_config0_full_parity(ws):
    w = synth.make_weights(0, 0, 0)
    g = GpuLayer(w, ws)
    g.check_weights()
    x = synth.make_activations(0, 0, 0, 8)
    g.check_forward(x)


@pytest.mark.parametrize("M,K,N,r", [
    (1, 64, 64, 16), (1, 512, 512, 32), (2, 100, 37, 8), (4, 1365, 130, 32), (8, 256, 192, 1),
    (16, 2048, 256, 64), (17, 320, 257, 24), (33, 1000, 66, 128), (48, 4096, 128, 48), (64, 704, 320, 128),
    (1, 11008, 256, 128), (5, 63, 1, 5), (40, 768, 200, 64), (41, 768, 200, 64),
])
def test_decode_shapes_parity(M, K, N, r, ws):
    c = synth.make_custom(1000 + M + K + N + r, M, K, N, r, act="student_t3")
    g = GpuLayer(c, ws)
    g.check_forward(c["x"])


@pytest.mark.parametrize("M,K,N,r", [
    (1, 8, 1, 1), (1, 128, 32, 16), (1, 4096, 1000, 64), (2, 4104, 96, 20), (3, 1024, 33, 128), (4, 12288, 160, 64),
    (4, 11008, 64, 128), (1, 3072, 3072, 32), (2, 768, 2304, 0), (4, 8, 130, 7), (1, 12288, 31, 128),
])
def test_few_token_single_launch_parity(M, K, N, r, ws):
    """M <= 4 with 16-byte rows takes the single persistent launch: tokens quantised inside
    the workgroups, partial sums of A x exchanged within the launch.  Afterwards the launch
    counter in the workspace has advanced by one, the arrival count is back at zero and no
    wait has run out; the two-launch path gives the same integers.  (Ranks that are not
    multiples of 8 have unaligned rows of B and take the two-launch path to begin with.)"""
    c = synth.make_custom(3000 + M + K + N + r, M, K, N, max(r, 1), act="student_t3")
    g = GpuLayer(c, ws, rank0=(r == 0))
    flags = lambda: ws.buf[:12].view(torch.int32).cpu().numpy().copy()
    for _ in range(3):
        before = flags()
        y1, _ = g.check_forward(c["x"])
        after = flags()
        assert after[0] == before[0] + (1 if r % 8 == 0 else 0) and after[1] == 0 and after[2] == 0, (before, after)
    hb.hgf_set_single_launch(0)
    try:
        before = flags()
        y2, _ = g.check_forward(c["x"])
        assert np.array_equal(flags(), before)
    finally:
        hb.hgf_set_single_launch(2)
    assert_close_fp16(y1, y2.astype(np.float64))


@pytest.mark.parametrize("M,K,N,r,path", [
    (65, 256, 128, 16, "direct"), (130, 512, 200, 32, "direct"), (256, 1365, 256, 64, "direct"),
    (1030, 256, 1500, 16, "prefill"), (800, 520, 2000, 64, "prefill"), (200, 1365, 7700, 32, "prefill"),
])
def test_large_m_parity(M, K, N, r, path, ws):
    c = synth.make_custom(2000 + M + K + N + r, M, K, N, r, act="student_t4")
    g = GpuLayer(c, ws)
    with path_taken(path):
        g.check_forward(c["x"])


@pytest.mark.parametrize("M,K,N,r", [(70, 4104, 96, 8), (66, 8200, 64, 16), (65, 16392, 40, 8)])
def test_large_m_long_rows_parity(M, K, N, r, ws):
    """Rows of 4104, 8200 and 16392 columns beyond 64 tokens, on the direct path: three, five and nine
    slices of d_in.  (The prefill path's quantiser at such rows, register depth by register depth:
    test_gpu_direct.test_prefill_path.)"""
    c = synth.make_custom(2100 + M + K + N + r, M, K, N, r, act="student_t4")
    g = GpuLayer(c, ws if K <= 11008 else hb.Workspace(M, K, 64, 128))
    with path_taken("direct"):
        g.check_forward(c["x"])


@pytest.mark.parametrize("M,path", [(150, "direct"), (3500, "prefill")])
def test_group_shares_one_launch(M, path, ws):
    """Four layers read slot 0.  At M = 3500 ranks 16, 24 and 32 pad to the same 32 columns of
    SiLU(A x), so their tiles (d_out 300, 256 and 40: two, one and one row tiles, the first and
    last ragged) go out as one launch of the prefill kernel; the rank-64 layer takes its own.  At
    M = 150 the direct path takes all four in one launch.  Each output is checked against the oracle
    and must equal, bit for bit, what the same layer gives on its own (on the same path)."""
    K = 384
    if M > 2048:
        ws = hb.Workspace(M, K, 300, 64)
    shapes = [(300, 16), (256, 24), (40, 32), (128, 64)]
    cases, layers = [], []
    slots = [None] * (len(shapes) + 1)
    for i, (N, r) in enumerate(shapes):
        c = synth.make_custom(7700 + i, M, K, N, r, act="student_t4", lora_std=0.05, w_std=0.05)
        if i == 0:
            x = c["x"]
            slots[0] = dev(x)
        g = GpuLayer(c, ws)
        g.layer.c.src_slot, g.layer.c.dst_slot = 0, i + 1
        cases.append(g)
        layers.append(g.layer)
        slots[i + 1] = torch.zeros((M, N), dtype=torch.float16, device="cuda")
    with path_taken(path):
        hb.hgf_stack_forward(hb.Stack(layers, slots, M), ws)
    torch.cuda.synchronize()
    for i, g in enumerate(cases):
        got = slots[i + 1].cpu().numpy()
        ref = g.oracle(x, dense=M > 2048)
        assert_close_fp16(got, ref["y"], f"layer {i}")
        with path_taken(path):
            y1, acc1 = g.forward(x)
        assert np.array_equal(acc1, ref["acc"])
        assert np.array_equal(got, y1), f"layer {i}: grouped launch and single layer differ"


@pytest.mark.parametrize("M", [12, 13, 33, 64])
def test_decode_group_with_many_row_blocks(M, ws):
    """Two layers read slot 0 and have 513 row-blocks between them (d_out 8200 and 8190, the
    last of either ragged; d_in 520: five k-tiles, the last ragged): one token group takes a row-block per
    workgroup with one tile in flight, 33 and 64 tokens (two groups) two row-blocks per workgroup, the
    last workgroup of the first layer with one.  Every output against the oracle, accumulators bit for bit
    against the single layer."""
    K = 520
    shapes = [(8200, 16), (8190, 40)]
    cases, layers = [], []
    slots = [None] * (len(shapes) + 1)
    for i, (N, r) in enumerate(shapes):
        c = synth.make_custom(7800 + i, M, K, N, r, act="student_t3", lora_std=0.05, w_std=0.05)
        if i == 0:
            x = c["x"]
            slots[0] = dev(x)
        g = GpuLayer(c, ws)
        g.layer.c.src_slot, g.layer.c.dst_slot = 0, i + 1
        cases.append(g)
        layers.append(g.layer)
        slots[i + 1] = torch.zeros((M, N), dtype=torch.float16, device="cuda")
    hb.hgf_stack_forward(hb.Stack(layers, slots, M), ws)
    torch.cuda.synchronize()
    for i, g in enumerate(cases):
        got = slots[i + 1].cpu().numpy()
        ref = g.oracle(x)
        assert_close_fp16(got, ref["y"], f"layer {i}")
        y1, acc1 = g.forward(x)
        assert np.array_equal(acc1, ref["acc"])
        assert_close_fp16(y1, ref["y"], f"layer {i} alone")


def test_gate_off_and_rank0_are_the_pure_ternary_layer(ws):
    c = synth.make_custom(77, 8, 512, 256, 32)
    full = GpuLayer(c, ws)
    y_full, ref = full.check_forward(c["x"])
    c_off = dict(c, alpha=np.zeros_like(c["alpha"]))
    y_off, _ = GpuLayer(c_off, ws).check_forward(c["x"])
    y_r0, _ = GpuLayer(c, ws, rank0=True).check_forward(c["x"])
    assert np.array_equal(y_off, y_r0)
    assert_close_fp16(y_r0, ref["y_tern"])
    assert not np.array_equal(y_full, y_r0)


def test_zero_token_and_extreme_accumulators(ws):
    K, N = 11008, 128
    W = np.full((N, K), 0.02, dtype=np.float32)
    W[1::2] *= -1                                       # rows alternate all +1 / all -1
    c = {"W": W, "d_in": K, "d_out": N, "rank": 0}
    g = GpuLayer(c, ws, rank0=True)
    x = np.full((3, K), 2.0, dtype=np.float16)
    x[1] = 0
    y, acc = g.forward(x)
    assert acc[0, 0] == 127 * K and acc[0, 1] == -127 * K and not acc[1].any() and not y[1].any()
    g.check_forward(x)


@pytest.mark.parametrize("M", [1, 2, 4, 8, 33, 100])
def test_tokens_of_fp16_subnormals(M, ws):
    """Tokens whose every value is an fp16 subnormal (below 6.1e-5), one of them below the
    quantiser's floor of 1e-5 for the absmax: the scale 127 / amax is then in the millions and the
    codes are only right if no stage flushes the subnormal inputs.  Through the single-layer entry
    point and as the first layer of a list (M <= 4: the whole-stack launch): the oracle's integers."""
    rng = np.random.default_rng(9100 + M)
    c = synth.make_custom(9100 + M, M, 520, 256, 16, lora_std=0.05, w_std=50.0)   # large s_w: outputs in fp16's normal range
    x = (rng.standard_normal((M, 520)) * 2e-5).clip(-6e-5, 6e-5).astype(np.float16)
    x[M // 2] = (rng.standard_normal(520) * 2e-6).astype(np.float16)       # absmax below the floor
    assert np.abs(x.astype(np.float32)).max() < 6.1e-5 and np.count_nonzero(x) > x.size // 2
    g = GpuLayer(c, ws)
    y, acc = g.forward(x)
    ref = g.oracle(x)
    assert np.abs(ref["acc"]).max() > 50
    assert np.array_equal(acc, ref["acc"])
    g.check_forward(x)
    c2 = synth.make_custom(9200 + M, M, 256, 128, 8, lora_std=0.05, w_std=0.05)
    g2 = GpuLayer(c2, ws)
    g.layer.c.src_slot, g.layer.c.dst_slot = 0, 1
    g2.layer.c.src_slot, g2.layer.c.dst_slot = 1, 2
    slots = [dev(x), torch.zeros((M, 256), dtype=torch.float16, device="cuda"),
             torch.zeros((M, 128), dtype=torch.float16, device="cuda")]
    hb.hgf_stack_forward(hb.Stack([g.layer, g2.layer], slots, M), ws)
    torch.cuda.synchronize()
    host = [t.cpu().numpy() for t in slots]
    assert_close_fp16(host[1], ref["y"], "first layer of the list")
    big = np.abs(ref["y"]) > 1e-4           # a wrong or flushed code moves these by percents
    assert big.mean() > 0.3
    assert np.all(np.abs(host[1].astype(np.float64) - ref["y"])[big] <= 5e-3 * np.abs(ref["y"])[big])
    assert np.all(np.abs(y.astype(np.float64) - ref["y"])[big] <= 5e-3 * np.abs(ref["y"])[big])
    assert_close_fp16(host[2], g2.oracle(host[1])["y"], "second layer of the list")


def test_repeated_calls_reuse_the_workspace(ws):
    """The workspace carries nothing from one call into the next: the same call twice, then a different
    shape, all on one workspace, give the oracle's integers every time."""
    a = synth.make_custom(5, 1, 4096, 512, 64)
    b = synth.make_custom(6, 16, 2048, 1024, 32)
    ga, gb = GpuLayer(a, ws), GpuLayer(b, ws)
    for _ in range(3):
        ga.check_forward(a["x"])
        gb.check_forward(b["x"])


# ------------------------------------------------------------------ stack

def _stack_case(cfg, M, ws, chained):
    wiring, inputs = synth.stack_wiring(cfg, chained=chained)
    cases, layers = [], []
    n_slots = 1 + max(w[3] for w in wiring)
    slots = [None] * n_slots
    for slot, layer in inputs.items():
        slots[slot] = dev(synth.make_activations(cfg, layer, 0, M))
    for (layer, proj, src, dst) in wiring:
        w = synth.make_weights(cfg, layer, proj)
        g = GpuLayer(w, ws)
        g.layer.c.src_slot, g.layer.c.dst_slot = src, dst
        cases.append(g)
        layers.append(g.layer)
        slots[dst] = torch.zeros((M, w["d_out"]), dtype=torch.float16, device="cuda")
    return cases, layers, slots, wiring


@pytest.mark.parametrize("chained", [False, True])
def test_config1_stack_teacher_forced(chained, ws):
    """The 8-layer, 56-linear decode stack at M=1 through hgf_stack_forward.  Every linear is
    checked against the oracle on the input the GPU actually gave it (the slot it read), so
    each of the 56 outputs meets the single-layer bar, and the single-layer entry point
    must reproduce the stack's bits.  Run twice: as the pure chain the benchmark times
    (its values shrink block by block: no norms or residuals between the linears), and
    with a fresh synthetic input per block so that every linear sees live activations."""
    cases, layers, slots, wiring = _stack_case(1, 1, ws, chained)
    st = hb.Stack(layers, slots, 1)
    flags = lambda: ws.buf[:32].view(torch.int32).cpu().numpy().copy()
    before = flags()
    hb.hgf_stack_forward(st, ws)
    torch.cuda.synchronize()
    after = flags()
    # the whole list ran as persistent launches over runs of layers (two: 48 layers fit one
    # launch's description), none of whose bounded waits ran out
    assert after[4] == before[4] + 2 and after[5] == 0 and after[2] == 0, (before, after)
    host = [s.cpu().numpy() for s in slots]
    live = 0
    for g, (_, _, src, dst) in zip(cases, wiring):
        ref = g.oracle(host[src])
        assert_close_fp16(host[dst], ref["y"], f"slot {dst}")
        y1, acc1 = g.forward(host[src])
        assert np.array_equal(y1, host[dst])
        assert np.array_equal(acc1, ref["acc"])
        live += int(np.abs(host[src].astype(np.float32)).max() > 1e-3 and np.abs(ref["acc"]).max() > 100)
    if not chained:
        assert live == len(wiring), live
    # the same list, one persistent launch per group of layers: the same integers, fp16 within a rounding
    hb.hgf_set_single_launch(1)
    try:
        for (_, _, _, dst) in wiring:
            slots[dst].zero_()
        hb.hgf_stack_forward(st, ws)
        torch.cuda.synchronize()
        assert np.array_equal(flags()[4:8], after[4:8])
        again = [s.cpu().numpy() for s in slots]
        if not chained:
            for (_, _, src, dst) in wiring:
                if np.array_equal(again[src], host[src]):
                    assert_close_fp16(again[dst], host[dst].astype(np.float64), f"slot {dst} (per-group launches)")
    finally:
        hb.hgf_set_single_launch(2)
    # end of the first block against the oracle's own chain (fp16 hand-over between layers)
    first = [i for i, w in enumerate(wiring) if w[0] == 0]
    chain = orc.stack_forward([{"T": cases[i].T_ref, "s_w": cases[i].s_w_ref, "A": cases[i].case["A"],
                                "B": cases[i].case["B"], "alpha": cases[i].case["alpha"]} for i in first],
                              [(wiring[i][2], wiring[i][3]) for i in first], host[0])
    end = wiring[first[-1]][3]
    ref_end = chain[end].astype(np.float64)
    rel = np.linalg.norm(host[end].astype(np.float64) - ref_end) / np.linalg.norm(ref_end)
    assert rel < 0.05, rel


@pytest.mark.parametrize("M", [1, 3, 4, 8, 16, 32, 40, 70, 3500])
def test_mixed_stack_teacher_forced(M, ws):
    """A short list that exercises the whole-stack launch and its fall-backs in one call: a
    group of two layers (one without correction), activations handed on inside the launch,
    ragged d_in (264), then a layer whose d_out (130) keeps it out of the whole-stack launch
    and one whose d_in (130) takes the two-launch path.  Every layer is checked against the
    oracle on the input the GPU gave it; a second run must reproduce the first bit for bit.
    M = 8 ... 70 take the direct path, whose prologue and grouped main kernel serve both layers of the
    group (one of them without correction) in one launch each.  M = 3500 sends the same list down
    the prefill path, whose preparation serves both layers of the group in one launch."""
    if M > 2048:
        ws = hb.Workspace(M, 512, 512, 32)
    shapes = [(256, 512, 16, 0, 1), (256, 384, 0, 0, 2), (512, 256, 32, 1, 3), (256, 264, 8, 3, 4),
              (264, 128, 24, 4, 5), (128, 130, 16, 5, 6), (130, 64, 8, 6, 7)]
    cases, layers = [], []
    slots = [None] * 8
    for i, (K, N, r, src, dst) in enumerate(shapes):
        c = synth.make_custom(7000 + 10 * M + i, M, K, N, max(r, 1), act="student_t4", lora_std=0.05, w_std=0.05)
        if i == 0:
            slots[0] = dev(c["x"])
        g = GpuLayer(c, ws, rank0=(r == 0))
        g.layer.c.src_slot, g.layer.c.dst_slot = src, dst
        cases.append(g)
        layers.append(g.layer)
        slots[dst] = torch.zeros((M, N), dtype=torch.float16, device="cuda")
    st = hb.Stack(layers, slots, M)
    flags = lambda: ws.buf[:32].view(torch.int32).cpu().numpy().copy()
    before = flags()
    with path_taken("prefill" if M > 2048 else "direct"):
        hb.hgf_stack_forward(st, ws)
    torch.cuda.synchronize()
    after = flags()
    assert after[4] == before[4] + (1 if M <= 4 else 0) and after[5] == 0 and after[2] == 0, (before, after)
    host = [s.cpu().numpy() for s in slots]
    for g, (K, N, r, src, dst) in zip(cases, shapes):
        ref = g.oracle(host[src], dense=M > 2048)
        assert_close_fp16(host[dst], ref["y"], f"slot {dst}")
        _, acc1 = g.forward(host[src])
        assert np.array_equal(acc1, ref["acc"])
    for (_, _, _, _, dst) in shapes:
        slots[dst].zero_()
    hb.hgf_stack_forward(st, ws)
    torch.cuda.synchronize()
    for (_, _, _, _, dst) in shapes:
        assert np.array_equal(slots[dst].cpu().numpy(), host[dst])


def test_stack_waits_give_up_and_recover(ws):
    """The give-up path of the whole-stack launch, forced from the host: with every wait between
    workgroups cut to one try, a chained list cannot hand its activations on in time.  The
    launch must still run to its end (no hang) and set the sticky error word; after
    hgf_workspace_init and with the default bound the same list gives the oracle's results."""
    M = 1
    shapes = [(512, 1024, 16, 0, 1), (1024, 512, 16, 1, 2), (512, 768, 32, 2, 3), (768, 256, 8, 3, 4)]
    cases, layers = [], []
    slots = [None] * 5
    for i, (K, N, r, src, dst) in enumerate(shapes):
        c = synth.make_custom(7700 + i, M, K, N, r, act="student_t4", lora_std=0.05, w_std=0.05)
        if i == 0:
            slots[0] = dev(c["x"])
        g = GpuLayer(c, ws)
        g.layer.c.src_slot, g.layer.c.dst_slot = src, dst
        cases.append(g)
        layers.append(g.layer)
        slots[dst] = torch.zeros((M, N), dtype=torch.float16, device="cuda")
    st = hb.Stack(layers, slots, M)
    flags = lambda: ws.buf[:32].view(torch.int32).cpu().numpy().copy()
    hb.hgf_workspace_init(ws)
    try:
        hb.hgf_set_wait_limit(1)
        hb.hgf_stack_forward(st, ws)
        torch.cuda.synchronize()                    # returns: every wait was bounded
    finally:
        hb.hgf_set_wait_limit(0)
    after = flags()
    assert after[2] != 0 and after[5] == 0, after   # error word set, every workgroup reached the end
    hb.hgf_workspace_init(ws)
    for (_, _, _, _, dst) in shapes:
        slots[dst].zero_()
    hb.hgf_stack_forward(st, ws)
    torch.cuda.synchronize()
    assert flags()[2] == 0
    host = [s_.cpu().numpy() for s_ in slots]
    for g, (K, N, r, src, dst) in zip(cases, shapes):
        assert_close_fp16(host[dst], g.oracle(host[src])["y"], f"slot {dst}")


# ------------------------------------------------------------------ full-size configurations, sampled

def _sampled(cfg, proj, M, ws, n_rows=96, n_tok=None):
    w = synth.make_weights(cfg, 0, proj)
    g = GpuLayer(w, ws)
    x = synth.make_activations(cfg, 0, proj, M)
    rng = np.random.default_rng(cfg * 100 + proj)
    rows = np.sort(rng.choice(w["d_out"], size=n_rows, replace=False))
    rows[0], rows[-1] = 0, w["d_out"] - 1
    tokens = None
    if n_tok is not None and n_tok < M:
        tokens = np.sort(rng.choice(M, size=n_tok, replace=False))
        tokens[0], tokens[-1] = 0, M - 1
    T = hb.hgf_unpack_weights(g.layer.packed, g.N, g.K).cpu().numpy()
    assert np.array_equal(T, g.T_ref)
    # sampled rows and tokens against the oracle's triple loop ...
    g.check_forward(x, rows=rows, tokens=tokens)
    # ... and EVERY accumulator and output against the oracle with the BLAS product in the
    # place of the loop (the CPU tests prove the two equal)
    y, acc = g.forward(x)
    ref = g.oracle(x, dense=True)
    assert np.array_equal(acc, ref["acc"]), "int32 accumulators differ from the oracle"
    assert_close_fp16(y, ref["y"])


@pytest.mark.parametrize("proj", [0, 4, 6])
@pytest.mark.parametrize("M", [1, 4, 16])
def test_config2_sampled(proj, M, ws):
    _sampled(2, proj, M, ws)


@pytest.mark.parametrize("proj,M", [(0, 1), (0, 64), (1, 8), (2, 1), (2, 32), (2, 64)])
def test_config4_sampled(proj, M, ws):
    _sampled(4, proj, M, ws)


@pytest.mark.parametrize("M", [1, 4])
def test_config4_stack_launch_sampled(M, ws):
    """The launch configuration the benchmark times, at full size: chained FFN blocks of
    config 4 through hgf_stack_forward, 18 blocks = 54 layers, which is one persistent
    launch over 16 blocks and a second over two.  (Every block uses the same three weight
    tensors: the launch does not know, and the oracle needs them only once.)  The first two
    blocks are checked layer by layer on sampled rows against the oracle on the input the GPU
    gave that layer.  Further down this chain without normalisation the activations grow
    beyond the configuration's distribution (absmax 170 at block 17 against 20 at the input),
    where an output that is a small difference of large terms misses a tolerance relative to
    the output alone on any path; there -- the end of the first launch and the second launch
    -- the oracle stays the reference with the relative part of the bound taken on
    |y_tern| + |g y_corr| (the two terms' own magnitudes, from the oracle), and every layer
    must also reproduce, bit for bit, what the single-layer entry point gives on that input."""
    n_blocks = 18
    wiring, _ = synth.stack_wiring(4, chained=True, n_layers=n_blocks)
    gl = [GpuLayer(synth.make_weights(4, 0, pi), ws) for pi in range(3)]
    slots = [None] * (1 + len(wiring))
    slots[0] = dev(synth.make_activations(4, 0, 0, M))
    layers = []
    for (_blk, pi, src, dst) in wiring:
        g = gl[pi]
        layers.append(hb.Layer(g.layer.packed, g.layer.s_w, g.N, g.K, g.layer.A, g.layer.B, g.layer.alpha,
                               src_slot=src, dst_slot=dst))
        slots[dst] = torch.zeros((M, g.N), dtype=torch.float16, device="cuda")
    st = hb.Stack(layers, slots, M)
    flags = lambda: ws.buf[:32].view(torch.int32).cpu().numpy().copy()
    before = flags()
    hb.hgf_stack_forward(st, ws)
    torch.cuda.synchronize()
    after = flags()
    assert after[4] == before[4] + 2 and after[5] == 0 and after[2] == 0, (before, after)
    rng = np.random.default_rng(4400 + M)
    for (blk, pi, src, dst) in wiring:
        if blk not in (0, 1, 15, 16, 17):
            continue
        g = gl[pi]
        x = slots[src].cpu().numpy()
        y = slots[dst].cpu().numpy()
        rows = np.sort(rng.choice(g.N, size=64, replace=False))
        rows[0], rows[-1] = 0, g.N - 1
        ref = g.oracle(x, rows)
        if blk <= 1:
            assert_close_fp16(y[:, rows], ref["y"], f"block {blk} projection {pi}")
        else:
            # the output is a difference of two large terms here: the relative part of the
            # bound is taken on the sum of their magnitudes, from the oracle's own two paths
            gate = np.abs(np.tanh(g.case["alpha"][rows].astype(np.float64)))[None, :]
            assert_close_fp16(y[:, rows], ref["y"], f"block {blk} projection {pi}",
                              scale=np.abs(ref["y_tern"]) + gate * np.abs(ref["y_corr"]))
        y1, _ = g.forward(x)
        assert np.array_equal(y, y1), f"block {blk} projection {pi}: whole-stack launch and single layer differ"


@pytest.mark.parametrize("proj", [0, 4, 6])
def test_config3_prefill_sampled(proj, ws):
    _sampled(3, proj, 2048, ws, n_rows=48, n_tok=24)


def _full_size_stack(cfg, M, ws):
    """One block of a configuration through hgf_stack_forward in the wiring the benchmark
    times (q, k, v share the block input; o reads v; up and gate read o; down reads up), so
    the grouped launches and their store paths run as they do there (no debug output).
    Every element of every layer's fp16 output is compared with the oracle evaluated on the
    input the GPU gave that layer (BLAS product in the place of the triple loop)."""
    cases, layers, slots, wiring = _stack_case(cfg, M, ws, chained=True)
    hb.hgf_stack_forward(hb.Stack(layers, slots, M), ws)
    torch.cuda.synchronize()
    assert ws.buf[:12].view(torch.int32).cpu().numpy()[2] == 0          # no bounded wait ran out
    host = [s.cpu().numpy() for s in slots]
    for g, (_, pi, src, dst) in zip(cases, wiring):
        ref = g.oracle(host[src], dense=True)
        assert np.abs(ref["acc"]).max() > 100, "dead input"
        assert_close_fp16(host[dst], ref["y"], f"config {cfg} projection {pi} (slot {dst})")
        rel = np.linalg.norm(host[dst].astype(np.float64) - ref["y"]) / np.linalg.norm(ref["y"])
        assert rel < 2e-3, (pi, rel)


def test_config3_stack_full_size_every_element(ws):
    _full_size_stack(3, 2048, ws)


@pytest.mark.parametrize("M", [1, 4, 16])
def test_config2_stack_full_size_every_element(M, ws):
    _full_size_stack(2, M, ws)


@pytest.mark.parametrize("M", [1, 8, 32, 64])
def test_config4_stack_full_size_every_element(M, ws):
    _full_size_stack(4, M, ws)


def test_mfma_rate_probe_runs_and_rejects_bad_arguments():
    """The measurement aid behind the prefill yardstick: a short run gives a plausible rate and
    clock; operand kinds outside 0..2 and iteration counts outside 1..2^20 are refused."""
    tops, ghz = hb.hgf_probe_mfma_rate(1, 50)
    assert 100.0 < tops < 6000.0, tops
    assert 0.5 < ghz < 3.0, ghz
    for kind, iters in ((3, 10), (-1, 10), (0, 0), (0, (1 << 20) + 1)):
        with pytest.raises(RuntimeError):
            hb.hgf_probe_mfma_rate(kind, iters)

