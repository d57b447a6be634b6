"""GPU parity of lpv_mask_topk against the float64 oracle.

The block scores are specified down to the summation order (float64, row-major
within a block, one addition after another), so the GPU's scores must equal
the oracle's bit for bit, and the kept set -- an integer decision taken from
them -- must be identical.
"""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl
from gpu_util import dev, say
from paper_2407_02068_amd import lpv

pytestmark = pytest.mark.gpu


def check(W, dtype, b_r, b_c, p, G=None, what=""):
    say("mask_topk", what, dtype, W.shape, (b_r, b_c), p, "taylor" if G is not None else "l2")
    m_gpu, s_gpu = lpv.mask_topk(dev(W, dtype), b_r, b_c, p,
                                 None if G is None else dev(G, dtype))
    torch.cuda.synchronize()
    m_ref, s_ref = oracle.block_mask(W, dtype, b_r, b_c, p, G)
    s = s_gpu.cpu().numpy()
    assert np.array_equal(s.view(np.uint64), s_ref.view(np.uint64)), "scores differ"
    m = m_gpu.cpu().numpy()
    assert np.array_equal(m, m_ref), "masks differ in %d blocks" % int((m != m_ref).sum())
    assert int(m.sum()) == oracle.keep_count(m.size, p)
    return m


def weights(seed, N, K, dtype, scale=0.02):
    g = np.random.default_rng(seed)
    return wl.quantize(g.normal(0, scale, (N, K)).astype(np.float32), dtype)


@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("b_r,b_c", [(16, 16), (32, 32), (64, 32), (16, 64)])
def test_scores_and_mask_match_oracle(dtype, b_r, b_c):
    W = weights(61 + b_r + b_c, 384, 256, dtype)
    G = weights(62 + b_r + b_c, 384, 256, dtype, scale=1.0)
    for p in (0, 30, 50, 90, 100):
        check(W, dtype, b_r, b_c, p, what="l2")
    check(W, dtype, b_r, b_c, 50, G, what="taylor")


def test_ties_go_to_the_lower_index():
    # equal blocks everywhere: the kept set is the first n_keep in row-major order
    W = np.ones((128, 192), np.float32)
    m = check(W, "f32", 32, 32, 40, what="all equal")
    n = oracle.keep_count(m.size, 40)
    assert m.reshape(-1)[:n].all() and not m.reshape(-1)[n:].any()
    # integer weights with many equal block sums
    g = np.random.default_rng(63)
    Wi = g.integers(-2, 3, (256, 256)).astype(np.float32)
    check(Wi, "f32", 16, 16, 50, what="integer ties")
    check(Wi.astype(np.float16), "f16", 16, 16, 75, Wi.astype(np.float16), what="integer taylor")


def test_headline_weight():
    # DeiT-B fc1: 3072 x 768 bf16 at 50%, and the 16x16 grid of the same weight
    W = wl.b_fc1().W
    check(W, "bf16", 32, 32, 50, what="b_fc1")
    check(W, "bf16", 16, 16, 75, what="b_fc1 16x16")


def test_mask_feeds_pack_and_linear():
    # the generated mask drives the hot path: pack it and check the layer
    w = wl.custom(64, 300, 384, 256, 32, 32, "bf16", "uniform", 50)
    m_gpu, _ = lpv.mask_topk(dev(w.W, "bf16"), 32, 32, 60)
    h = lpv.bsr_pack(dev(w.W, "bf16"), m_gpu, 32, 32)
    Y = lpv.bsr_linear(h, dev(w.X, "bf16"), dev(w.bias, "bf16"))
    torch.cuda.synchronize()
    mask, _ = oracle.block_mask(w.W, "bf16", 32, 32, 60)
    r = oracle.linear(w.X, w.W, "bf16", 32, 32, mask, w.bias)
    err = oracle.rel_err(Y.float().cpu().numpy().astype(np.float64), r)
    say("  mask -> pack -> linear rel err %.3e" % err)
    assert err <= 2e-2


def test_unaligned_weight_rows():
    # row strides that are not multiples of 16 bytes (a view one element into
    # a wider buffer): the scores take the kernel that reads element by element
    for dtype in ("bf16", "f32"):
        W = weights(65, 192, 256, dtype)
        G = weights(66, 192, 256, dtype, scale=1.0)
        say("mask_topk unaligned rows", dtype)
        for taylor in (False, True):
            buf = torch.zeros((192, 257), dtype=dev(W, dtype).dtype, device="cuda")
            buf[:, 1:] = dev(W, dtype)
            gbuf = torch.zeros_like(buf)
            gbuf[:, 1:] = dev(G, dtype)
            m_gpu, s_gpu = lpv.mask_topk(buf[:, 1:], 32, 32, 50, gbuf[:, 1:] if taylor else None)
            torch.cuda.synchronize()
            m_ref, s_ref = oracle.block_mask(W, dtype, 32, 32, 50, G if taylor else None)
            assert np.array_equal(s_gpu.cpu().numpy().view(np.uint64), s_ref.view(np.uint64))
            assert np.array_equal(m_gpu.cpu().numpy(), m_ref)


def test_many_blocks_with_ties():
    # 12288 blocks (more than the 8192 that are ranked: the radix selection) of small
    # integers, so many block scores are equal: ties still go to the lower index
    g = np.random.default_rng(67)
    Wi = g.integers(-2, 3, (2048, 1536)).astype(np.float32)
    for p in (25, 50, 90):
        check(Wi, "f32", 16, 16, p, what="12288 integer blocks")
    Gi = g.integers(-2, 3, (2048, 1536)).astype(np.float32)
    check(Wi.astype(np.float16), "f16", 16, 16, 50, Gi.astype(np.float16), what="12288 taylor")


@pytest.mark.parametrize("N,K", [(16, 16 * 9), (2048, 1024), (128, 8208)])
def test_ranking_with_ties_across_chunks(N, K):
    # up to 8192 blocks every block is ranked, 4096 keys at a time and 8 blocks per
    # workgroup: 9 blocks, two whole chunks, one chunk and 8 more
    g = np.random.default_rng(68)
    Wi = g.integers(-1, 2, (N, K)).astype(np.float32)
    for p in (1, 50, 97):
        check(Wi, "f32", 16, 16, p, what="integer blocks")
    check(np.ones_like(Wi), "f32", 16, 16, 37, what="equal blocks")


def test_ranking_of_equal_blocks_takes_no_longer():
    # 32768 blocks, ranked for the delta curve: scores all different, and all equal
    t = []
    for W in (torch.randn((8192, 1024), device="cuda"), torch.ones((8192, 1024), device="cuda")):
        ms = []
        for _ in range(9):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            lpv.delta_curve(W, W, W[:0].reshape(0, 8192, 1024), 16, 16, 0.0, [0, 50, 100])
            e1.record()
            torch.cuda.synchronize()
            ms.append(e0.elapsed_time(e1))
        t.append(sorted(ms)[4])
    say("ranking 32768 blocks: different %.3f ms, equal %.3f" % tuple(t))
    assert t[1] <= 1.3 * t[0]
