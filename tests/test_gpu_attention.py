"""GPU parity of the differential-attention decode step against the CPU oracle (fp64): fp16 outputs
within 2e-3 + 1e-2 |o| over head sizes 8 .. 128, ragged cache lengths (one position, chunk
boundaries, an empty sequence), several sequences, and the shapes of the paper's own model
(d = 512, 8 heads: q, k 16 heads of 32 columns, v 8 heads of 32) and of a 7B-shape one."""
import numpy as np
import pytest
import torch

from oracle import hgf_oracle as orc
from paper_2602_05269_amd import binding as hb
from parity import assert_close_fp16, dev

pytestmark = pytest.mark.gpu


def _case(seed, B, L, H, d, scale=1.0):
    rng = np.random.default_rng(seed)
    q = (scale * rng.standard_normal((B, 2 * H, d))).astype(np.float16)
    k = (scale * rng.standard_normal((B, L, 2 * H, d))).astype(np.float16)
    v = rng.standard_normal((B, L, H, d)).astype(np.float16)
    return q, k, v


@pytest.mark.parametrize("B,L,H,d,lens", [
    (1, 1, 1, 8, [1]), (2, 37, 3, 16, [37, 11]), (3, 300, 2, 32, [256, 257, 1]), (2, 512, 8, 32, [512, 100]),
    (2, 700, 4, 64, [700, 0]), (1, 1024, 2, 128, [1000]), (4, 130, 5, 64, [130, 129, 128, 2]),
])
def test_diff_attention_decode_parity(B, L, H, d, lens):
    q, k, v = _case(B * 1000 + L + H + d, B, L, H, d)
    lam = orc.diff_attention_lambda_init(2 * d)
    out = hb.hgf_diff_attention_decode(dev(q), dev(k), dev(v), dev(np.array(lens, dtype=np.int32)), lam)
    torch.cuda.synchronize()
    ref = orc.diff_attention_decode(q, k, v, lens, lam)
    assert_close_fp16(out.cpu().numpy(), ref, "attention output")
    assert np.abs(ref).max() > 1e-2


def test_diff_attention_peaked_scores_and_cache_beyond_len_ignored():
    """Large scores (a softmax close to one-hot, where the chunk maxima differ widely) and
    garbage behind lens in the caches: rows past the length must not matter, NaNs included."""
    B, L, H, d = 2, 600, 2, 32
    q, k, v = _case(5, B, L, H, d, scale=3.0)
    lens = [300, 513]
    for b, n in enumerate(lens):
        k[b, n:] = np.float16(np.nan)
        v[b, n:] = np.float16(np.inf)
    out = hb.hgf_diff_attention_decode(dev(q), dev(k), dev(v), dev(np.array(lens, dtype=np.int32)), 0.5)
    torch.cuda.synchronize()
    ref = orc.diff_attention_decode(q, k, v, lens, 0.5)
    assert_close_fp16(out.cpu().numpy(), ref, "attention output")


def test_diff_attention_model_shapes():
    # the paper's model: d = 512, 8 heads -> q, k: 16 heads of 32; v: 8 heads of 32; context 512
    q, k, v = _case(11, 4, 512, 8, 32)
    lens = [512, 400, 17, 256]
    lam = orc.diff_attention_lambda_init(64)
    out = hb.hgf_diff_attention_decode(dev(q), dev(k), dev(v), dev(np.array(lens, dtype=np.int32)), lam)
    assert_close_fp16(out.cpu().numpy(), orc.diff_attention_decode(q, k, v, lens, lam))
    # a 7B-shape block: d = 4096, 32 heads -> q, k: 64 heads of 64; v: 32 heads of 64; 4096 cached positions
    q, k, v = _case(12, 1, 4096, 32, 64)
    out = hb.hgf_diff_attention_decode(dev(q), dev(k), dev(v), dev(np.array([4096], dtype=np.int32)), 0.8)
    assert_close_fp16(out.cpu().numpy(), orc.diff_attention_decode(q, k, v, [4096], 0.8))


@pytest.mark.parametrize("d,L,lens", [(8, 16700, [16385, 16384, 16700]), (32, 17000, [17000, 1, 65])])
def test_diff_attention_many_chunks(d, L, lens):
    # more chunks of 256 positions than one batch of the merge (64), and wavefronts of 64 positions that are empty
    q, k, v = _case(d + L, len(lens), L, 1, d)
    out = hb.hgf_diff_attention_decode(dev(q), dev(k), dev(v), dev(np.array(lens, dtype=np.int32)), 0.8)
    assert_close_fp16(out.cpu().numpy(), orc.diff_attention_decode(q, k, v, lens, 0.8))


@pytest.mark.parametrize("d,L,lens", [(8, 256, [256, 0, 65]), (64, 200, [0, 200, 1]), (128, 257, [257, 0, 256]), (32, 1100, [769, 1024, 1025]),
                                      (128, 900, [900, 768, 1]), (64, 900, [3, 900, 513])])
def test_diff_attention_few_chunks(d, L, lens):
    # one chunk (no merging launch), two, five, four (heads fastest); empty sequences
    q, k, v = _case(d + L, len(lens), L, 3, d)
    out = hb.hgf_diff_attention_decode(dev(q), dev(k), dev(v), dev(np.array(lens, dtype=np.int32)), 0.8)
    assert_close_fp16(out.cpu().numpy(), orc.diff_attention_decode(q, k, v, lens, 0.8))


def test_diff_attention_cache_of_more_chunks_than_a_narrow_grid_extent():
    # a cache of 65537 chunks (one more than a grid's second extent takes), nearly all of it empty
    L = 65536 * 256 + 1
    q, k, v = _case(77, 1, 300, 1, 8)
    kc = torch.zeros((1, L, 2, 8), dtype=torch.float16, device="cuda")
    vc = torch.zeros((1, L, 1, 8), dtype=torch.float16, device="cuda")
    kc[:, :300], vc[:, :300] = dev(k), dev(v)
    out = hb.hgf_diff_attention_decode(dev(q), kc, vc, torch.tensor([300], dtype=torch.int32, device="cuda"), 0.8)
    assert_close_fp16(out.cpu().numpy(), orc.diff_attention_decode(q, k, v, [300], 0.8))


def test_diff_attention_many_workgroups():
    # 64 columns, five chunks, more than 2048 workgroups: chunks fastest; few of them: heads fastest
    q, k, v = _case(78, 26, 1030, 16, 64)
    lens = [1030, 1024, 1025, 1, 0, 700] * 4 + [255, 256]
    out = hb.hgf_diff_attention_decode(dev(q), dev(k), dev(v), dev(np.array(lens, dtype=np.int32)), 0.8).cpu().numpy()
    assert_close_fp16(out, orc.diff_attention_decode(q, k, v, lens, 0.8))
    few = hb.hgf_diff_attention_decode(dev(q[:2]), dev(k[:2]), dev(v[:2]), dev(np.array(lens[:2], dtype=np.int32)), 0.8)
    assert np.array_equal(few.cpu().numpy(), out[:2])


def test_diff_attention_rejects_bad_arguments():
    lib = hb.lib()
    assert lib.hgf_diff_attention_workspace_bytes(1, 128, 4, 24) == 0          # d_h not a power of two
    assert lib.hgf_diff_attention_workspace_bytes(1, 128, 4, 256) == 0
    assert lib.hgf_diff_attention_workspace_bytes(1, 1 << 20, 64, 128) == 0    # a sequence's cache beyond 2 GiB
    assert lib.hgf_diff_attention_decode(None, 0x100, 0x100, 0x100, 1, 8, 1, 8, 0.5, 0x100, 0x100, 1 << 20, None) == 1
    assert lib.hgf_diff_attention_decode(0x100, 0x100, 0x100, 0x100, 1, 8, 1, 12, 0.5, 0x100, 0x100, 1 << 20, None) == 2
    assert lib.hgf_diff_attention_decode(0x100, 0x104, 0x100, 0x100, 1, 8, 1, 8, 0.5, 0x100, 0x100, 1 << 20, None) == 3
    assert lib.hgf_diff_attention_decode(0x100, 0x100, 0x100, 0x100, 1, 8, 1, 8, 0.5, 0x100, 0x100, 16, None) == 5
