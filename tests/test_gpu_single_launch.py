"""GPU parity of one group of up to four tokens in the persistent launch: base-3 weights on either side of its rule,
tokens quantised together (tokens with infinities and NaN among them), workgroups that compute the sums they wait for
themselves (base-3), and outputs that lie over the tokens (two launches).  Accumulators bit for bit, outputs within
2e-3 + 1e-2 |y| (fp16 rounding of h and y)."""
import numpy as np
import pytest
import torch

from paper_2602_05269_amd import binding as hb
from paper_2602_05269_amd import synth
from parity import GpuLayer, assert_close_fp16, dev
from test_gpu_b3 import B3Layer

pytestmark = pytest.mark.gpu


def launches(ws):
    torch.cuda.synchronize()
    return int(ws.buf[:4].view(torch.int32).cpu()[0])


@pytest.mark.parametrize("M,K,N,r,one", [
    # the rule's edges: columns, whole 16-byte pieces, the longest row, tokens
    (1, 768, 33, 16, True), (1, 760, 33, 16, False), (2, 1536, 95, 32, True), (2, 1528, 95, 32, False), (1, 2004, 64, 8, False),
    (1, 12288, 31, 128, True), (1, 12296, 31, 128, False), (2, 12288, 40, 64, True), (3, 4096, 64, 16, False),
    # a row's last k-tile: whole, one byte of its first half, its second half; fewer k-tiles than wavefronts; rank 0
    (1, 1120, 64, 24, True), (2, 4008, 65, 40, True), (1, 1048, 1, 0, True), (2, 2000, 257, 0, True),
    # two units of rows per workgroup
    (2, 1600, 8300, 16, True),
    # more than 2048 rows
    (1, 1528, 2049, 16, False), (1, 1528, 2048, 16, True), (1, 1536, 2049, 16, True), (2, 1592, 2049, 16, False), (2, 1536, 2048, 16, True),
])
def test_base3_in_the_persistent_launch(M, K, N, r, one):
    c = synth.make_custom(9800 + M + K + N + r, M, K, N, max(r, 1), act="student_t3", lora_std=0.05)
    ws = hb.Workspace(M, K, N, r)
    before = launches(ws)
    B3Layer(c, ws, rank0=r == 0).check_forward(c["x"], ws, dense=True)
    assert (launches(ws) != before) == one


@pytest.mark.parametrize("M,K,N,r", [(2, 64, 33, 16), (3, 3584, 95, 40), (4, 3592, 64, 128), (4, 12288, 31, 16), (3, 7176, 70, 0)])
@pytest.mark.parametrize("bad", [None, np.inf, np.nan])
def test_tokens_quantised_together(M, K, N, r, bad):
    c = synth.make_custom(9900 + M + K + N, M, K, N, max(r, 1), act="student_t3", lora_std=0.05)
    x = c["x"].copy()
    x[1] = 0                                # (its scale is the smallest there is)
    ws = hb.Workspace(M, K, N, r)
    g = GpuLayer(c, ws, rank0=r == 0)
    if bad is None:
        y, acc = g.forward(x)
        ref = g.oracle(x, dense=True)
        assert np.array_equal(acc, ref["acc"]), "int32 accumulators differ from the oracle"
        assert_close_fp16(y, ref["y"])
        return
    x[0, K // 2] = bad
    x[M - 1, K - 1] = -bad
    before = launches(ws)
    y, acc = g.forward(x)
    assert launches(ws) != before
    hb.hgf_set_single_launch(0)
    try:
        y2, acc2 = g.forward(x)
    finally:
        hb.hgf_set_single_launch(2)
    assert np.array_equal(acc, acc2)
    assert np.array_equal(np.isnan(y), np.isnan(y2))
    fine = np.isfinite(y2)
    assert_close_fp16(y[fine], y2[fine])


@pytest.mark.parametrize("M,K,N,r", [(2, 11008, 64, 100), (1, 4096, 300, 128), (1, 1000, 9000, 24), (1, 1600, 9000, 24)])
def test_base3_workgroups_that_wait_help_themselves(M, K, N, r):
    c = synth.make_custom(9950 + M + K, M, K, N, r, act="student_t3", lora_std=0.05)
    ws = hb.Workspace(M, K, N, r)
    g, f = B3Layer(c, ws), hb.hgf_linear_forward_b3
    x = dev(c["x"])
    want = f(x, g.layer, ws).cpu()
    try:
        hb.hgf_set_wait_limit(1)
        for _ in range(3):
            assert torch.equal(f(x, g.layer, ws).cpu(), want)
    finally:
        hb.hgf_set_wait_limit(0)
    assert torch.equal(f(x, g.layer, ws).cpu(), want)
    assert int(ws.buf[8:12].view(torch.int32).cpu()[0]) == 0


@pytest.mark.parametrize("M,K,N,r,b3", [(1, 4096, 4096, 64, False), (2, 2048, 2048, 16, True), (3, 1024, 2000, 0, False)])
def test_output_over_the_tokens(M, K, N, r, b3):
    c = synth.make_custom(9970 + M + K, M, K, N, max(r, 1), act="student_t3", lora_std=0.05)
    ws = hb.Workspace(M, K, N, r)
    g = (B3Layer if b3 else GpuLayer)(c, ws, rank0=r == 0)
    f = hb.hgf_linear_forward_b3 if b3 else hb.hgf_linear_forward
    x = dev(c["x"])
    want = f(x, g.layer, ws).cpu().numpy()
    both = torch.zeros(M * max(K, N), dtype=torch.float16, device="cuda")
    tokens, y = both[:M * K].view(M, K), both[:M * N].view(M, N)
    tokens.copy_(x)
    before = launches(ws)
    f(tokens, g.layer, ws, y=y)
    assert launches(ws) == before
    assert_close_fp16(y.cpu().numpy(), want)
