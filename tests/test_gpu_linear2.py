"""GPU parity of pq_linear2 (two weight matrices on the same tokens, gate and up of an MLP block).

Against the oracle: the layer's gate of the other tests (codes differ from the oracle's only at rounding ties,
the oracle's product and epilogue on the GPU's codes reproduce both outputs within one fp16 ulp).  Against
pq_linear: outputs bit-identical to two separate calls, in the fused single launch (few tokens; one row
group may start in the first matrix and the next in the second, matrices of different heights, with and
without rotation) and in the quantize-once + two products form (more tokens).
"""

import numpy as np
import pytest

import oracle as O
import small_tiles as T
from paper_2410_05265_amd import synth
from pq_testlib import check_end_to_end, dev, host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pq():
    import paper_2410_05265_amd.binding as b
    b.lib()
    return b


def layer(M, K, Na, Nb, h, seed):
    x = synth.activations(M, K, seed)
    sx = O.calibrate_absmax(synth.calibration(K, seed), h)
    wa, swa = O.weight_rtn(synth.weights(Na, K, seed))
    wb, swb = O.weight_rtn(synth.weights(Nb, K, seed + 1))
    return x, sx, O.pack(wa), swa, O.pack(wb), swb


# (M, K, N_a, N_b, had_block): one token to a small prefill; heights that make 1, 2 or 4 rows per wavefront;
# N_a not a multiple of the rows a workgroup takes at a time; 5 tokens and 64 tokens leave the fused launch; the last
# row: both products in one launch of small tiles, of several sizes, the second matrix taller or a single ragged tile
CASES = [(1, 512, 256, 256, 1), (1, 4096, 1008, 528, 1), (2, 2048, 4096, 2064, 128), (4, 1024, 16, 8192, 64),
         (1, 8192, 14336, 14336, 1), (3, 4096, 9008, 9008, 4096), (1, 14336, 2048, 1040, 128),
         (1, 4096, 14336, 14336, 1),      # gate and up of Llama-3-8B at one token: the launch bench.py times

         (5, 1024, 528, 272, 128), (64, 1024, 528, 272, 1), (16, 4096, 1024, 512, 128),
         (24, 4096, 272, 1040, 1), (40, 1152, 4240, 16, 128), (100, 640, 48, 8208, 1), (300, 384, 2064, 2064, 1)]


@pytest.mark.parametrize("M,K,Na,Nb,h", CASES)
def test_two_matrices_one_quantization(pq, M, K, Na, Nb, h):
    x, sx, wa, swa, wb, swb = layer(M, K, Na, Nb, h, seed=M + K + Na)
    dx, dwa, dswa, dwb, dswb = dev(x), dev(wa), dev(swa), dev(wb), dev(swb)
    oa, ob, ws = pq.pq_linear2(dx, dwa, dswa, dwb, dswb, float(sx), h)
    codes = host(ws)[: M * K // 2].reshape(M, K // 2)
    check_end_to_end(x, wa, swa, sx, h, host(oa), codes)
    check_end_to_end(x, wb, swb, sx, h, host(ob), codes)
    ra, _ = pq.pq_linear(dx, dwa, dswa, float(sx), h)
    rb, wsb = pq.pq_linear(dx, dwb, dswb, float(sx), h)
    assert np.array_equal(host(oa).view(np.uint16), host(ra).view(np.uint16))
    assert np.array_equal(host(ob).view(np.uint16), host(rb).view(np.uint16))
    assert np.array_equal(codes, host(wsb)[: M * K // 2].reshape(M, K // 2))


@pytest.mark.parametrize("M,K,Na,Nb,h", [(70, 1152, 272, 528, 128), (300, 512, 896, 256, 1), (33, 4096, 64, 512, 4096)])
def test_two_matrices_prepacked(pq, M, K, Na, Nb, h):
    """pq_linear2_f6: the outputs of two pq_linear_f6 calls, and of pq_linear2 on the canonical weights, bit for bit."""
    x, sx, wa, swa, wb, swb = layer(M, K, Na, Nb, h, seed=M + K)
    dx, dwa, dswa, dwb, dswb = dev(x), dev(wa), dev(swa), dev(wb), dev(swb)
    ta, tb = pq.pq_repack_f6(dwa), pq.pq_repack_f6(dwb)
    oa, ob, _ = pq.pq_linear2_f6(dx, ta, dswa, tb, dswb, float(sx), h)
    ra, _ = pq.pq_linear_f6(dx, ta, dswa, float(sx), h)
    rb, _ = pq.pq_linear_f6(dx, tb, dswb, float(sx), h)
    ca, cb, _ = pq.pq_linear2(dx, dwa, dswa, dwb, dswb, float(sx), h)
    for got, one, canon in ((oa, ra, ca), (ob, rb, cb)):
        assert np.array_equal(host(got).view(np.uint16), host(one).view(np.uint16))
        assert np.array_equal(host(got).view(np.uint16), host(canon).view(np.uint16))


# equal heights: one launch for both (256-wide tiles in one and in several rounds, 384, 512, the mix of 512 and 384, a last
# tile that is ragged in both directions), every small tile among them
@pytest.mark.parametrize("M,K,N", [(1030, 256, 4096), (2048, 128, 8208), (2048, 128, 6144), (4000, 256, 2064), (2000, 128, 14336), (40, 640, 272), (300, 384, 1040)] +
                         [(M, K, N) for _, M, N, K in T.TWO_PREPACKED])
def test_two_matrices_of_one_height_prepacked(pq, M, K, N):
    x = dev(synth.activations(M, K, seed=M + K))
    ws = [dev(synth.random_packed(N, K, seed=N + i, stream=7)) for i in (0, 1)]
    steps = [dev(synth.random_scales(N, seed=N + i)) for i in (0, 1)]
    tiles = [pq.pq_repack_f6(w) for w in ws]
    a, b, work = pq.pq_linear2_f6(x, tiles[0], steps[0], tiles[1], steps[1], 0.21, 1)
    xq = pq.pq_rotate_quant(x, 1, 0.21)
    for got, w, s in ((a, ws[0], steps[0]), (b, ws[1], steps[1])):
        want, _ = pq.pq_w4a4_gemm(xq, w, s, 0.21)
        assert np.array_equal(host(got).view(np.uint16), host(want).view(np.uint16))
    # forced widths take the same launch
    for tile in (2, 3, 4):
        prev = pq.pq_set_gemm_f6_tile(tile)
        try:
            fa, fb, _ = pq.pq_linear2_f6(x, tiles[0], steps[0], tiles[1], steps[1], 0.21, 1)
        finally:
            pq.pq_set_gemm_f6_tile(prev)
        assert np.array_equal(host(fa).view(np.uint16), host(a).view(np.uint16))
        assert np.array_equal(host(fb).view(np.uint16), host(b).view(np.uint16))


@pytest.mark.parametrize("tile,M,Na,Nb,K", T.TWO_PACKED)
def test_two_packed_products_of_every_small_tile(pq, tile, M, Na, Nb, K):
    """One launch of small tiles against the tiled kernel's products of the same codes, bit for bit."""
    assert pq.pq_gemm_small_tile(M, Na, Nb, K) == tile
    x = dev(synth.activations(M, K, seed=M + K))
    ws = [dev(synth.random_packed(N, K, seed=N + i, stream=7)) for i, N in enumerate((Na, Nb))]
    steps = [dev(synth.random_scales(N, seed=N + i)) for i, N in enumerate((Na, Nb))]
    a, b, _ = pq.pq_linear2(x, ws[0], steps[0], ws[1], steps[1], 0.21, 1)
    xq = pq.pq_rotate_quant(x, 1, 0.21)
    prev = pq.pq_set_gemm_variant(2)
    try:
        for got, w, s in ((a, ws[0], steps[0]), (b, ws[1], steps[1])):
            want, _ = pq.pq_w4a4_gemm(xq, w, s, 0.21)
            assert np.array_equal(host(got).view(np.uint16), host(want).view(np.uint16))
    finally:
        pq.pq_set_gemm_variant(prev)


def test_argument_errors(pq):
    import torch
    x, sx, wa, swa, wb, swb = layer(1, 512, 32, 32, 1, seed=3)
    dx, dwa, dswa, dwb, dswb = dev(x), dev(wa), dev(swa), dev(wb), dev(swb)
    with pytest.raises(Exception):
        pq.pq_linear2(dx, dwa, dswa, dwb[:24], dswb[:24], float(sx), 1)          # N_b not a multiple of 16
    with pytest.raises(Exception):
        pq.pq_linear2(dx, dwa, dswa, dwb, dswb, float(sx), 1, workspace=torch.empty(16, dtype=torch.uint8, device="cuda"))
    with pytest.raises(Exception):
        pq.pq_linear2(dx, dwa, dswa, dwb, dswb, 0.0, 1)
