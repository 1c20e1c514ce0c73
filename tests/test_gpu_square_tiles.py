"""Every near-square tile of the prepacked product, on one matrix and on two: outputs bit for bit those of a forced width of the other
kernel, and sampled sums those of the oracle.  Rows and channels end inside a tile, inside a 32-row image and, where a
wavefront has an odd count of operands, inside a pair of them; one round of tiles and several, full tiles among them; outputs in
ordinary stores and past the memory-side cache, in whole lines, halves and smaller pieces."""

import numpy as np
import pytest
import torch

import oracle as O
from pq_testlib import host
from square_tiles import ONE, STREAM_ONE, STREAM_TWO, TWO      # (which take their tiles: test_launches.py)

pytestmark = pytest.mark.gpu


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


@pytest.mark.parametrize("_,M,N,K", ONE + STREAM_ONE)
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


@pytest.mark.parametrize("_,M,N,K", TWO + STREAM_TWO)
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


@pytest.mark.parametrize("start", [0, 8, 16, 32, 64])
def test_outputs_that_start_within_a_line(start):
    """start: fp16 values before the output, with guards on either side."""
    import paper_2410_05265_amd.binding as pq
    M, N, K = 2319, 10048, 1024
    gen = torch.Generator(device="cuda").manual_seed(5)
    x6, w6 = (pq.pq_repack_f6(codes(r, K, gen)) for r in (M, N))
    sw = torch.rand((N,), device="cuda", generator=gen) * 0.02 + 1e-3
    guard = torch.full((M * N + 128,), 7.0, dtype=torch.float16, device="cuda")
    out = guard[start:start + M * N].view(M, N)
    pq.pq_w4a4_gemm_f6(x6, w6, sw, 0.0917, M, N, K, out=out)
    want, _ = forced(pq, lambda: pq.pq_w4a4_gemm_f6(x6, w6, sw, 0.0917, M, N, K))
    assert torch.equal(out, want) and bool((guard[:start] == 7.0).all()) and bool((guard[start + M * N:] == 7.0).all())
