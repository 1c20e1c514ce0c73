"""The product of int8 activations on tiles of 64, 96, 128, 160 and 192 tokens x 128 channels: last tiles with one row and one
group of 16 channels, one stage, odd and even counts of them, more tiles than the chip has CUs, runs of K in planes (an
automatic split gets scratch memory for 16 planes), and the tiles of 32 x 32 results that the plan still takes.  Integer sums are exact; both epilogues are within an fp16 ulp."""

import numpy as np
import pytest
import torch

import oracle as O
from paper_2410_05265_amd import synth
from pq_testlib import dev, host, ulp_diff
from tile_plans import BYTES

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pq():
    import paper_2410_05265_amd.binding as b
    b.lib()
    return b


# (which tile each of these takes: test_tile_plans.py)
@pytest.mark.parametrize("M,N,K,planes", [c[1:] for c in BYTES])
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
