"""Every tile size of the packed product: outputs bit for bit those of tiles of 128 x 128, with a static step, a step per token and a
zero point, and sampled sums those of the oracle.  Rows and channels end inside a tile and inside a wavefront's 32 x 32 results; fewer
stages than the ring holds and more; one round of tiles and two."""

import numpy as np
import pytest
import torch

import oracle as O
from packed_tiles import TILES      # (which take their tiles: test_launches.py)
from pq_testlib import host


@pytest.mark.gpu
@pytest.mark.parametrize("_,M,N,K", TILES)
def test_tile(_, M, N, K):
    import paper_2410_05265_amd.binding as pq
    gen = torch.Generator(device="cuda").manual_seed(M)
    x, w = (torch.randint(0, 256, (r, K // 2), dtype=torch.uint8, device="cuda", generator=gen) for r in (M, N))
    x[M - 1] = 0x88                                                # the largest sums: -8 with -8
    w[N - 1] = 0x88
    sw, srow = (torch.rand((n,), device="cuda", generator=gen) * 0.02 + 1e-3 for n in (N, M))
    zc = torch.randint(-3000, 3000, (N,), dtype=torch.int32, device="cuda", generator=gen)

    def results():
        guard = torch.full((M + 1, N), 7.0, dtype=torch.float16, device="cuda")
        got = [*pq.pq_w4a4_gemm(x, w, sw, 0.0917, want_acc=True), pq.pq_gemm_dynamic(x, 4, w, sw, srow)[0], pq.pq_w4a4_gemm_zp(x, w, sw, 0.0917, zc)[0]]
        pq.pq_w4a4_gemm(x, w, sw, 0.0917, out=guard[:M])
        assert torch.equal(guard[:M], got[0]) and bool((guard[M] == 7.0).all())
        return got

    variant = pq.pq_set_gemm_variant(2)                            # the tiled kernel
    try:
        got = results()
        saved = pq.pq_set_gemm_tile(2)
        try:
            want = results()
        finally:
            pq.pq_set_gemm_tile(saved)
    finally:
        pq.pq_set_gemm_variant(variant)
    assert all(torch.equal(a, b) for a, b in zip(got, want))
    rows, cols = np.unique(np.r_[0:M:97, M - 1]), np.unique(np.r_[0:N:131, N - 1])
    assert np.array_equal(host(got[1])[np.ix_(rows, cols)].astype(np.int64), O.gemm_i64(O.unpack(host(x[rows])), O.unpack(host(w[cols]))))
