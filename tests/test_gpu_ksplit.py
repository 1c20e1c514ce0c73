"""GPU parity of the small-tile products that split K over a workgroup's wavefronts (outputs of few tiles).

Accumulators are exact integers whatever the order of the partial sums, so they equal the oracle's, and the fp16
outputs equal those of the large-tile kernels bit for bit.  Shapes: every tile size the rule picks (small_tiles.py), among
them fewer stages than wavefronts (most wavefronts then add zeros), stage counts the wavefronts do not share evenly (the
prologue and the tails of the two-stage ring), rows that end in the middle of a stage, and the longest row.
"""

import numpy as np
import pytest

import oracle as O
import small_tiles as T
from paper_2410_05265_amd import synth
from pq_testlib import dev, host, ulp_diff

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pq():
    import paper_2410_05265_amd.binding as b
    b.lib()
    return b


def operands(M, N, K):
    return (synth.random_packed(M, K, seed=M + K), synth.random_packed(N, K, seed=N + K, stream=7),
            synth.random_scales(N, seed=N), np.float32(0.2173))


@pytest.mark.parametrize("tile,M,N,K", T.ONE_PREPACKED)
def test_prepacked_product(pq, tile, M, N, K):
    assert pq.pq_gemm_small_tile(M, N, 0, K, prepacked=True) == tile
    xq, wq, sw, sx = operands(M, N, K)
    x6, w6 = pq.pq_repack_f6(dev(xq)), pq.pq_repack_f6(dev(wq))
    acc_ref = O.gemm_i64(O.unpack(xq), O.unpack(wq))
    out, acc = pq.pq_w4a4_gemm_f6(x6, w6, dev(sw), float(sx), M, N, K, want_acc=True)
    assert np.array_equal(host(acc).astype(np.int64), acc_ref)
    assert ulp_diff(host(out), O.epilogue(acc_ref, sx, sw)).max() <= 1
    prev = pq.pq_set_gemm_f6_tile(2)
    try:
        big, _ = pq.pq_w4a4_gemm_f6(x6, w6, dev(sw), float(sx), M, N, K)
    finally:
        pq.pq_set_gemm_f6_tile(prev)
    assert np.array_equal(host(big).view(np.uint16), host(out).view(np.uint16))
    # each output alone
    only, none = pq.pq_w4a4_gemm_f6(x6, w6, dev(sw), float(sx), M, N, K)
    assert none is None and np.array_equal(host(only).view(np.uint16), host(out).view(np.uint16))
    none, only = pq.pq_w4a4_gemm_f6(x6, w6, dev(sw), float(sx), M, N, K, want_out=False, want_acc=True)
    assert none is None and np.array_equal(host(only), host(acc))


def forced(pq, variant, fn, *a, **kw):
    prev = pq.pq_set_gemm_variant(variant)
    try:
        return fn(*a, **kw)
    finally:
        pq.pq_set_gemm_variant(prev)


@pytest.mark.parametrize("tile,M,N,K", T.ONE_PACKED)
def test_packed_product_with_every_epilogue(pq, tile, M, N, K):
    assert pq.pq_gemm_small_tile(M, N, 0, K) == tile
    xq, wq, sw, sx = operands(M, N, K)
    x, w, s = dev(xq), dev(wq), dev(sw)
    acc_ref = O.gemm_i64(O.unpack(xq), O.unpack(wq))
    out, acc = pq.pq_w4a4_gemm(x, w, s, float(sx), want_acc=True)
    assert np.array_equal(host(acc).astype(np.int64), acc_ref)
    assert ulp_diff(host(out), O.epilogue(acc_ref, sx, sw)).max() <= 1
    tiled, _ = forced(pq, 2, pq.pq_w4a4_gemm, x, w, s, float(sx))
    assert np.array_equal(host(tiled).view(np.uint16), host(out).view(np.uint16))
    none, only = pq.pq_w4a4_gemm(x, w, s, float(sx), want_out=False, want_acc=True)
    assert none is None and np.array_equal(host(only), host(acc))
    # the tokens' own steps
    srow = dev((0.05 + 0.4 * np.random.default_rng(M).random(M)).astype(np.float32))
    dyn, acc = pq.pq_gemm_dynamic(x, 4, w, s, srow, want_acc=True)
    tiled, _ = forced(pq, 2, pq.pq_gemm_dynamic, x, 4, w, s, srow)
    assert np.array_equal(host(acc).astype(np.int64), acc_ref)
    assert np.array_equal(host(tiled).view(np.uint16), host(dyn).view(np.uint16))
    # a zero-point's per-channel integers
    corr = pq.pq_zero_point_correction(w, 3)
    zp, acc = pq.pq_w4a4_gemm_zp(x, w, s, float(sx), corr, want_acc=True)
    tiled, _ = forced(pq, 2, pq.pq_w4a4_gemm_zp, x, w, s, float(sx), corr)
    assert np.array_equal(host(acc).astype(np.int64), acc_ref)
    assert np.array_equal(host(tiled).view(np.uint16), host(zp).view(np.uint16))


def test_packed_extreme_codes_on_the_longest_row(pq):
    """All codes -8 at the largest K: the int32 sums of 256 acc hold 256 * 64 * K."""
    M, N, K = 40, 64, 130944
    x, w = (dev(np.full((r, K // 2), 0x88, dtype=np.uint8)) for r in (M, N))
    sw = synth.random_scales(N, seed=1)
    out, acc = pq.pq_w4a4_gemm(x, w, dev(sw), 1e-5, want_acc=True)
    assert (host(acc) == 64 * K).all()
    assert ulp_diff(host(out), O.epilogue(np.full((M, N), 64 * K, dtype=np.int64), np.float32(1e-5), sw)).max() <= 1


def test_limits_of_the_per_token_form_stay(pq):
    """Rows longer than 65536 channels were refused with per-token steps and still are."""
    import torch
    K = 65536 + 128
    x, w = (torch.zeros((r, K // 2), dtype=torch.uint8, device="cuda") for r in (40, 64))
    with pytest.raises(RuntimeError, match="PQ_ERR_UNSUPPORTED"):
        pq.pq_gemm_dynamic(x, 4, w, torch.ones(64, device="cuda"), torch.ones(40, device="cuda"))


def test_prepacked_extreme_codes_on_the_longest_row(pq):
    """All codes -8 at the largest K: every partial sum and the total stay exact in fp32 (below 2^24)."""
    M, N, K = 40, 64, 262016                     # the largest multiple of 128 the product accepts
    x6 = pq.pq_repack_f6(dev(np.full((M, K // 2), 0x88, dtype=np.uint8)))
    w6 = pq.pq_repack_f6(dev(np.full((N, K // 2), 0x88, dtype=np.uint8)))
    sw = synth.random_scales(N, seed=1)
    out, acc = pq.pq_w4a4_gemm_f6(x6, w6, dev(sw), 1e-5, M, N, K, want_acc=True)
    assert (host(acc) == 64 * K).all()
    assert ulp_diff(host(out), O.epilogue(np.full((M, N), 64 * K, dtype=np.int64), np.float32(1e-5), sw)).max() <= 1
