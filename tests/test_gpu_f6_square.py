"""The 256 x 256 tiles that the prepacked product takes for long rows and large operands: the automatic choice against a forced width of the other
kernel, whole outputs bit for bit, and sampled rows and channels against the oracle's integer sums.  Rows and channels end
inside a tile and inside a 32-row image, with an odd count of 256-channel pairs, and with two rounds of tiles."""

import numpy as np
import pytest
import torch

import oracle as O
from pq_testlib import host
from tile_plans import SQUARE

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", SQUARE)            # (which take them: test_tile_plans.py)
def test_square_tiles_match_the_other_kernel_and_the_oracle(M, N, K):
    import paper_2410_05265_amd.binding as pq
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M)
    x, w = (torch.randint(0, 256, (r, K // 2), dtype=torch.uint8, device="cuda", generator=gen) for r in (M, N))
    x[M - 1] = 0x88                                                # the largest sums: -8 with -8
    w[N - 1] = 0x88
    sw = torch.rand((N,), device="cuda", generator=gen) * 0.02 + 1e-3
    x6, w6 = pq.pq_repack_f6(x), pq.pq_repack_f6(w)
    out, acc = pq.pq_w4a4_gemm_f6(x6, w6, sw, 0.0917, M, N, K, want_acc=True)
    alone, _ = pq.pq_w4a4_gemm_f6(x6, w6, sw, 0.0917, M, N, K)
    saved = pq.pq_set_gemm_f6_tile(4)
    try:
        want_out, want_acc = pq.pq_w4a4_gemm_f6(x6, w6, sw, 0.0917, M, N, K, want_acc=True)
    finally:
        pq.pq_set_gemm_f6_tile(saved)
    assert torch.equal(acc, want_acc) and torch.equal(out, want_out) and torch.equal(alone, out)
    rows, cols = np.unique(np.r_[0:M:97, M - 1]), np.unique(np.r_[0:N:131, N - 1])
    ref = O.gemm_i64(O.unpack(host(x[rows])), O.unpack(host(w[cols])))
    assert np.array_equal(host(acc)[np.ix_(rows, cols)].astype(np.int64), ref)
