"""The product of int8 activations on tiles of 64, 96, 128, 160 and 192 tokens x 128 channels: last tiles with one row and one
group of 16 channels, one stage, odd and even counts of them, more tiles than the chip has CUs, and runs of K in planes (an
automatic split gets scratch memory for 16 planes).  Integer sums are exact; both epilogues are within an fp16 ulp."""

import numpy as np
import pytest
import torch

import oracle as O
from paper_2410_05265_amd import synth
from pq_testlib import dev, host, ulp_diff

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pq():
    import paper_2410_05265_amd.binding as b
    b.lib()
    return b


# (the height that the estimates choose is given beside each shape; 64 also where everything fits one tile)
@pytest.mark.parametrize("M,N,K,planes", [(33, 16, 128, 0), (65, 144, 256, 0), (129, 272, 1152, 0),               # 64
                                          (1441, 2032, 384, 0),                                                # 96
                                          (897, 4016, 128, 0), (1000, 4080, 256, 0),                           # 128
                                          (2081, 2064, 384, 0),                                                # 160
                                          (1345, 4016, 640, 0), (1475, 4080, 128, 0),                          # 192
                                          (70, 272, 4096, 16), (135, 3600, 6400, 16), (390, 2576, 12288, 16)])  # 64, 96, 128, split
def test_tile_heights_edges_and_runs(pq, M, N, K, planes):
    q = synth.random_codes(M, K, seed=M, stream=9, lo=-128, hi=127)
    q[0], q[-1] = -128, 127                                       # the largest sums
    wq, sw, srow = synth.random_packed(N, K, seed=N, stream=7), synth.random_scales(N, seed=7), synth.random_scales(M, seed=8)
    ref = O.gemm_i64(q, O.unpack(wq))
    xq = dev(O.group_even_odd(q))
    ws = torch.empty(planes * M * N * 4, dtype=torch.uint8, device="cuda") if planes else None
    out, acc = pq.pq_w4a8_gemm(xq, dev(wq), dev(sw), 0.013, want_acc=True, workspace=ws)
    outd, accd = pq.pq_gemm_dynamic(xq, 8, dev(wq), dev(sw), dev(srow), want_acc=True, workspace=ws)
    alone, _ = pq.pq_w4a8_gemm(xq, dev(wq), dev(sw), 0.013, workspace=ws)
    assert np.array_equal(host(acc).astype(np.int64), ref) and np.array_equal(host(accd).astype(np.int64), ref)
    assert ulp_diff(host(out), O.epilogue(ref, np.float32(0.013), sw)).max() <= 1
    assert ulp_diff(host(outd), O.epilogue(ref, srow, sw)).max() <= 1
    assert torch.equal(out, alone)
