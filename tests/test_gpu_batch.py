"""GPU parity of the task queue (a list of five phases or more for 5 to 16 tokens in one launch): every layer
equals, bit for bit, what two launches per group give, and the oracle's result within 2e-3 + 1e-2 |y|.  The
launch counter of the queue is int32 word 8 of the workspace, its workgroup count and next task are words 9
and 11 (zero between launches), word 2 is the sticky error."""
import numpy as np
import pytest
import torch

from paper_2602_05269_amd import binding as hb
from paper_2602_05269_amd import synth
from parity import GpuLayer, assert_close_fp16, dev

pytestmark = pytest.mark.gpu


def _flags(ws):
    return ws.buf[:64].view(torch.int32).cpu().numpy().copy()


def _list(shapes, M, ws, x=None, dst_of=None):
    """shapes: (d_in, d_out, rank, source slot, destination slot); slot 0 holds the tokens."""
    cases, layers, slots = [], [], {}
    for i, (K, N, r, src, dst) in enumerate(shapes):
        c = synth.make_custom(9300 + 10 * M + i, M, K, N, max(r, 1), act="student_t4", lora_std=0.05, w_std=0.05)
        if i == 0:
            slots[0] = dev(c["x"] if x is None else x(c["x"]))
        g = GpuLayer(c, ws, rank0=r == 0)
        g.layer.c.src_slot, g.layer.c.dst_slot = src, dst
        cases.append(g)
        layers.append(g.layer)
        slots.setdefault(dst, torch.zeros((M, N), dtype=torch.float16, device="cuda"))
    slots = [slots[i] for i in range(1 + max(slots))]
    return cases, hb.Stack(layers, slots, M), slots


def _run(st, slots, ws, level):
    for s in slots[1:]:
        s.fill_(float("nan"))
    hb.hgf_set_single_launch(level)
    try:
        hb.hgf_stack_forward(st, ws)
    finally:
        hb.hgf_set_single_launch(2)
    torch.cuda.synchronize()
    return [s.cpu().numpy() for s in slots]


# long enough rows (beyond 2048 columns or 32 ranks) to be no short rows
CHAIN = [(2056, 2304, 40, 0, 1), (2056, 2080, 0, 0, 2), (2304, 4104, 64, 1, 3), (2304, 33, 128, 1, 4), (4104, 2112, 8, 3, 5),
         (4104, 2056, 16, 3, 6), (4104, 95, 0, 3, 7), (2112, 8184, 128, 5, 8), (8184, 1160, 24, 8, 9), (2056, 2304, 48, 6, 10)]


@pytest.mark.parametrize("M", [5, 8, 9, 16])
def test_queue_equals_two_launches_and_the_oracle(M):
    """Ragged rows and columns, ranks past 64 and none, groups of one to three layers, one to four slices of A x,
    a group that reads an older slot than the last; three times over one workspace."""
    ws = hb.Workspace(M, 8184, 8184, 128)
    cases, st, slots = _list(CHAIN, M, ws)
    two = _run(st, slots, ws, 0)
    before = _flags(ws)
    for _ in range(3):
        one = _run(st, slots, ws, 2)
        for i, (a, b) in enumerate(zip(one, two)):
            assert np.array_equal(a.view(np.uint16), b.view(np.uint16)), f"slot {i}"
    after = _flags(ws)
    assert after[8] == before[8] + 3 and after[9] == 0 and after[11] == 0 and after[2] == 0, (before, after)
    for g, (K, N, r, src, dst) in zip(cases, CHAIN):
        ref = g.oracle(one[src], dense=True)
        # The chain has no norms and grows, and an output may be a small difference of large terms B h, each of which
        # carries the rounding of h to fp16 (2^-11 of it) and of its fp32 sum: 2^-10 of the sum of their magnitudes
        # is allowed beside 1e-2 |y|.
        scale = np.abs(ref["y"])
        if r:
            c = g.case
            v = one[src].astype(np.float64) @ c["A"].astype(np.float64).T
            gate = np.abs(np.tanh(c["alpha"].astype(np.float64)))[None, :]
            scale = scale + 2.0 ** -10 / 1e-2 * gate * (np.abs(v / (1 + np.exp(-v))) @ np.abs(c["B"].astype(np.float64)).T)
        assert_close_fp16(one[dst], ref["y"], f"slot {dst}", scale=scale)


@pytest.mark.parametrize("M", [7, 16])
def test_queue_of_many_row_blocks(M):
    """Two, three and four row-blocks per task, more tasks than compute units, a layer boundary inside a task."""
    shapes = [(2056, 16000, 8, 0, 1), (2056, 8000, 40, 0, 2), (2056, 12000, 40, 0, 3), (8000, 2056, 8, 2, 4), (2056, 33000, 0, 4, 5),
              (2056, 2080, 64, 4, 6), (2080, 9001, 40, 6, 7), (2080, 5000, 40, 6, 8), (5000, 64, 8, 8, 9)]
    ws = hb.Workspace(M, 8000, 33000, 64)
    _, st, slots = _list(shapes, M, ws)
    two = _run(st, slots, ws, 0)
    before = _flags(ws)
    one = _run(st, slots, ws, 2)
    assert _flags(ws)[8] > before[8]
    for i, (a, b) in enumerate(zip(one, two)):
        assert np.array_equal(a.view(np.uint16), b.view(np.uint16)), f"slot {i}"


@pytest.mark.parametrize("bad", [np.inf, np.nan])
def test_queue_with_an_odd_token(bad):
    def spoil(x):
        x = x.copy()
        x[1, 3] = bad
        return x

    M = 6
    ws = hb.Workspace(M, 8184, 8184, 128)
    _, st, slots = _list(CHAIN, M, ws, x=spoil)
    two, one = _run(st, slots, ws, 0), _run(st, slots, ws, 2)
    for i, (a, b) in enumerate(zip(one, two)):
        assert np.array_equal(np.isnan(a), np.isnan(b)) and np.array_equal(a[~np.isnan(a)], b[~np.isnan(b)]), f"slot {i}"


def test_queue_and_reused_slots():
    """A list that writes its slots again and again (no two of its outputs may change places), and one over the
    input's own slot: launches end where memory is written a second time."""
    M, d = 8, 2056
    ws = hb.Workspace(M, d, d, 48)
    shapes = [(d, d, 48, 0, 1), (d, d, 48, 1, 2), (d, d, 48, 2, 3), (d, d, 48, 3, 4), (d, d, 48, 4, 5), (d, d, 48, 5, 6), (d, d, 48, 6, 1),
              (d, d, 48, 1, 2), (d, d, 48, 2, 0), (d, d, 48, 0, 3), (d, d, 48, 3, 4), (d, d, 48, 4, 5), (d, d, 48, 5, 6)]
    _, st, slots = _list(shapes, M, ws)
    x = slots[0].clone()
    two = _run(st, slots, ws, 0)
    before = _flags(ws)
    for _ in range(2):
        slots[0].copy_(x)
        one = _run(st, slots, ws, 2)
        for i, (a, b) in enumerate(zip(one, two)):
            assert np.array_equal(a.view(np.uint16), b.view(np.uint16)), f"slot {i}"
    assert _flags(ws)[8] > before[8]


def test_queue_shares_a_workspace_and_a_graph():
    """Whole-stack launches for four tokens and queues in turn over one workspace; the queue captured in a graph
    and replayed between eager calls: always the same bits."""
    ws = hb.Workspace(16, 8184, 8184, 128)
    _, st16, s16 = _list(CHAIN, 16, ws)
    _, st4, s4 = _list([(2056, 2304, 40, 0, 1), (2304, 4104, 64, 1, 2), (4104, 2112, 8, 2, 3)], 4, ws)
    want16, want4 = _run(st16, s16, ws, 2), _run(st4, s4, ws, 2)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        hb.hgf_stack_forward(st16, ws)
    for _ in range(4):
        for s in s16[1:]:
            s.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert all(np.array_equal(a.cpu().numpy().view(np.uint16), b.view(np.uint16)) for a, b in zip(s16, want16))
        assert all(np.array_equal(a, b) for a, b in zip(_run(st4, s4, ws, 2), want4))
        assert all(np.array_equal(a.view(np.uint16), b.view(np.uint16)) for a, b in zip(_run(st16, s16, ws, 2), want16))
    assert _flags(ws)[2] == 0


class _ShiftedWorkspace:
    """A workspace that starts 16 bytes (all that is asked of it) past a multiple of 256."""

    def __init__(self, shift, *dims):
        self.bytes = hb.hgf_workspace_bytes(*dims)
        whole = torch.zeros(self.bytes + 512, dtype=torch.uint8, device="cuda")
        start = -whole.data_ptr() % 256 + shift
        self.buf = whole[start:start + self.bytes]
        hb.hgf_workspace_init(self)


@pytest.mark.parametrize("shift", [16, 112, 240])
def test_queue_in_a_workspace_between_two_lines(shift):
    """Other tokens in every pass over one workspace: nothing of a pass before is taken for a token of this one."""
    M, d = 8, 2304
    ws = _ShiftedWorkspace(shift, M, d, d, 48)
    _, st, slots = _list([(d, d, 48, i, i + 1) for i in range(8)], M, ws)
    x = slots[0].clone()
    for seed in range(3):
        slots[0].copy_(x.roll(seed, 0) * (1.0 - 0.25 * seed))
        two = _run(st, slots, ws, 0)
        before = _flags(ws)
        one = _run(st, slots, ws, 2)
        assert _flags(ws)[8] == before[8] + 1
        for i, (a, b) in enumerate(zip(one, two)):
            assert np.array_equal(a.view(np.uint16), b.view(np.uint16)), f"slot {i}"


@pytest.mark.parametrize("M", [8, 16])
def test_queue_gives_up_without_a_wrong_number(M):
    """Every wait bounded by one try, set from the host: the launch ends, the sticky word is set, and an output is
    what it should be or NaN, layers without ranks (whose quantiser passes over a NaN) among them."""
    ws = hb.Workspace(M, 8184, 8184, 128)
    shapes = CHAIN[:8] + [(8184, 2304, 0, 8, 9), (2304, 2080, 48, 9, 10)]
    _, st, slots = _list(shapes, M, ws)
    want = _run(st, slots, ws, 2)
    assert _flags(ws)[2] == 0
    try:
        hb.hgf_set_wait_limit(1)
        got = _run(st, slots, ws, 2)
    finally:
        hb.hgf_set_wait_limit(0)
    after = _flags(ws)
    assert after[2] != 0 and after[9] == 0 and after[11] == 0, after
    for i, (a, b) in enumerate(zip(got, want)):
        fine = ~np.isnan(a)
        assert np.array_equal(a[fine].view(np.uint16), b[fine].view(np.uint16)), f"slot {i}"
    assert np.isnan(got[-1]).all()
    hb.hgf_workspace_init(ws)
    for a, b in zip(_run(st, slots, ws, 2), want):
        assert np.array_equal(a.view(np.uint16), b.view(np.uint16))
    assert _flags(ws)[2] == 0


@pytest.mark.parametrize("M,shapes", [
    # rows of 8192 columns at 16 tokens have room for two layers of 64 ranks, not of 128: each phase for itself
    (16, [(2056, 8192, 64, 0, 1), (8192, 4200, 64, 1, 2), (8192, 4200, 64, 1, 3), (4200, 2056, 128, 2, 4), (2056, 2056, 40, 4, 5),
          (2056, 2056, 40, 5, 6)]),
    # a group of more rows than a phase has words for ends a run, it does not undo it
    (5, [(2056, 2056, 48, i, i + 1) for i in range(5)] + [(2056, 40000, 8, 5, 6), (2056, 40000, 8, 5, 7)]),
])
def test_one_phase_does_not_cost_a_list_its_queue(M, shapes):
    ws = hb.Workspace(M, 8192, 40000, 128)
    _, st, slots = _list(shapes, M, ws)
    two = _run(st, slots, ws, 0)
    before = _flags(ws)
    one = _run(st, slots, ws, 2)
    assert _flags(ws)[8] == before[8] + 1
    for i, (a, b) in enumerate(zip(one, two)):
        assert np.array_equal(a.view(np.uint16), b.view(np.uint16)), f"slot {i}"


def test_blocks_that_reuse_their_slots():
    """Every block writes the same q, k, v, o, up, gate and down slots: no run is long enough for the queue, and every
    output is that of level 0."""
    M, d, f = 8, 2304, 2400
    ws = hb.Workspace(M, f, f, 48)
    block = [(d, d, 48, 0, 1), (d, d, 48, 0, 2), (d, d, 48, 0, 3), (d, d, 48, 1, 4), (d, f, 48, 4, 5), (d, f, 48, 4, 6), (f, d, 48, 5, 0)]
    _, st, slots = _list(block * 3, M, ws)
    x = slots[0].clone()
    two = _run(st, slots, ws, 0)
    for _ in range(2):
        slots[0].copy_(x)
        for i, (a, b) in enumerate(zip(_run(st, slots, ws, 2), two)):
            assert np.array_equal(a.view(np.uint16), b.view(np.uint16)), f"slot {i}"
    assert _flags(ws)[8] == 0 and _flags(ws)[2] == 0


def _chain(n, d, r, slot=0, first=1):
    """n groups, each of which reads the one before, from `slot` on; outputs in slots from `first` on."""
    return [(d, d, r, slot if i == 0 else first + i - 1, first + i) for i in range(n)]


@pytest.mark.parametrize("shapes,queues", [
    (_chain(6, 2304, 48), 0),
    (_chain(5, 2304, 48) + [(2304, 2304, 48, 1, 6)], 0),
    (_chain(5, 2304, 48) + [(2304, 2304, 48, 1, 6), (2304, 2304, 48, 2, 7)], 1),
    (_chain(5, 2304, 48) + _chain(2, 2304, 48, 0, 6), 1),
    (_chain(17, 2304, 48), 0),
    (_chain(16, 2304, 48) + [(2304, 2304, 48, 0, 17), (2304, 2304, 48, 1, 18), (2304, 2304, 48, 2, 19), (2304, 2304, 48, 3, 20),
                             (2304, 2304, 48, 4, 21)], 1),
])
def test_chains_take_two_launches_per_group(shapes, queues):
    """A run that is one chain of groups is left to two launches each, with the bits of the queue; one with two groups
    beside the chain is not, also where it begins behind a longer chain."""
    M = 8
    ws = hb.Workspace(M, 2304, 2304, 48)
    _, st, slots = _list(shapes, M, ws)
    queue = _run(st, slots, ws, 2)
    before = _flags(ws)
    got = _run(st, slots, ws, 3)
    assert _flags(ws)[8] == before[8] + queues
    for i, (a, b) in enumerate(zip(got, queue)):       # (a long chain may grow past the largest fp16)
        assert np.array_equal(a, b, equal_nan=True), f"slot {i}"


def test_a_chain_of_more_weights_than_caches_hold_takes_the_queue():
    """256 MiB of distinct weights; the same chain over one layer's weights takes two launches per group."""
    M, d, n = 5, 8192, 16
    ws = hb.Workspace(M, d, d, 0)
    gen = torch.Generator(device="cuda").manual_seed(5)
    packed = [hb.hgf_quantize_pack_weights(torch.randn((d, d), generator=gen, device="cuda") * 0.02, ws) for _ in range(n)]
    x = torch.randn((M, d), generator=gen, device="cuda").half()
    for same in (False, True):
        slots = [x] + [torch.empty((M, d), dtype=torch.float16, device="cuda") for _ in range(n)]
        layers = [hb.Layer(*packed[0 if same else i], d, d, src_slot=i, dst_slot=i + 1) for i in range(n)]
        st = hb.Stack(layers, slots, M)
        want = _run(st, slots, ws, 0)
        before = _flags(ws)
        got = _run(st, slots, ws, 3)
        assert _flags(ws)[8] == before[8] + (0 if same else 1)
        for i, (a, b) in enumerate(zip(got, want)):
            assert np.array_equal(a.view(np.uint16), b.view(np.uint16)), f"slot {i}"
