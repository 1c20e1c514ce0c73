"""Every near-square tile of the prepacked product, on one matrix and on two: outputs bit for bit those of a forced width of the other
kernel, and sampled sums those of the oracle.  Rows and channels end inside a tile, inside a 32-row image and, where a
wavefront has an odd count of operands, inside a pair of them; one round of tiles and several, full tiles among them."""

import ctypes

import numpy as np
import pytest
import torch

import oracle as O
from pq_testlib import host

# tile (10 * operands of 16 tokens + of 16 channels per wavefront), tokens, channels out, channels in
ONE = [(44, 129, 12208, 1024), (46, 294, 11408, 1024), (48, 1543, 9872, 1024), (58, 1358, 12368, 1024), (64, 270, 11152, 1280),
       (66, 1797, 8752, 1024), (68, 2738, 7248, 1024), (78, 2349, 10032, 1024), (87, 1948, 12304, 1024), (88, 2468, 12816, 1024)]
TWO = [(44, 68, 8368, 1024), (46, 259, 6096, 1024), (48, 2858, 2576, 1024), (58, 591, 13168, 1024), (64, 132, 9040, 1024),
       (66, 651, 11280, 1024), (68, 1471, 6576, 1024), (78, 1538, 7312, 1024), (87, 1156, 9872, 1024), (88, 2922, 4720, 1024)]


def tile(pq, M, N, K, two):
    rule = pq.lib()["_ZN2pq20gemm_f6_takes_squareElllb"]      # (pq::gemm_f6_takes_square: the launch's own rule)
    rule.restype, rule.argtypes = ctypes.c_int, [ctypes.c_int64] * 3 + [ctypes.c_bool]
    return rule(M, N, K, two)


@pytest.mark.parametrize("two,cases", [(False, ONE), (True, TWO)])
def test_every_tile_has_its_shape(two, cases):
    import paper_2410_05265_amd.binding as pq
    assert [tile(pq, M, N, K, two) for _, M, N, K in cases] == [c[0] for c in cases]
    assert all(M % 32 and N % 32 for _, M, N, _ in cases)


def codes(rows, K, gen):
    q = torch.randint(0, 256, (rows, K // 2), dtype=torch.uint8, device="cuda", generator=gen)
    q[rows - 1] = 0x88                                             # the largest sums: -8 with -8
    return q


def forced(pq, call):
    saved = pq.pq_set_gemm_f6_tile(2)
    try:
        return call()
    finally:
        pq.pq_set_gemm_f6_tile(saved)


@pytest.mark.gpu
@pytest.mark.parametrize("_,M,N,K", ONE)
def test_one_matrix(_, M, N, K):
    import paper_2410_05265_amd.binding as pq
    gen = torch.Generator(device="cuda").manual_seed(M)
    x, w = codes(M, K, gen), codes(N, K, gen)
    sw = torch.rand((N,), device="cuda", generator=gen) * 0.02 + 1e-3
    x6, w6 = pq.pq_repack_f6(x), pq.pq_repack_f6(w)
    out, acc = pq.pq_w4a4_gemm_f6(x6, w6, sw, 0.0917, M, N, K, want_acc=True)
    alone, _ = pq.pq_w4a4_gemm_f6(x6, w6, sw, 0.0917, M, N, K)
    want_out, want_acc = forced(pq, lambda: pq.pq_w4a4_gemm_f6(x6, w6, sw, 0.0917, M, N, K, want_acc=True))
    assert torch.equal(acc, want_acc) and torch.equal(out, want_out) and torch.equal(alone, out)
    rows, cols = np.unique(np.r_[0:M:97, M - 1]), np.unique(np.r_[0:N:131, N - 1])
    assert np.array_equal(host(acc)[np.ix_(rows, cols)].astype(np.int64), O.gemm_i64(O.unpack(host(x[rows])), O.unpack(host(w[cols]))))


@pytest.mark.gpu
@pytest.mark.parametrize("_,M,N,K", TWO)
def test_two_matrices(_, M, N, K):
    import paper_2410_05265_amd.binding as pq
    gen = torch.Generator(device="cuda").manual_seed(M)
    x = torch.randn((M, K), device="cuda", generator=gen).half()
    w6 = [pq.pq_repack_f6(codes(N, K, gen)) for _ in range(2)]
    sw = [torch.rand((N,), device="cuda", generator=gen) * 0.02 + 1e-3 for _ in range(2)]
    guard = [torch.full((M + 1, N), 7.0, dtype=torch.float16, device="cuda") for _ in range(2)]
    pq.pq_linear2_f6(x, w6[0], sw[0], w6[1], sw[1], 0.31, 1, out_a=guard[0][:M], out_b=guard[1][:M])
    want = forced(pq, lambda: [pq.pq_linear_f6(x, w6[i], sw[i], 0.31, 1)[0] for i in range(2)])
    for i in range(2):
        assert torch.equal(guard[i][:M], want[i]) and bool((guard[i][M] == 7.0).all())
