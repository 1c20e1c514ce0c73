"""The layer of 5 to 16 tokens without rotation in one launch (and of two matrices from 2 tokens on): codes and outputs are those
of the quantizer launch and the tiled product, bit for bit.  The shapes, and that they take this launch: fused_shapes.py, test_launches.py.

A second matrix starts inside a task; token counts are odd and even.  Inputs: values on rounding ties of the step and one fp16 step beside
them, infinities, NaN, zeros and subnormals.
"""

import numpy as np
import pytest
import torch

import fused_shapes
import oracle as O
from paper_2410_05265_amd import synth
from pq_testlib import check_end_to_end, dev, host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pq():
    import paper_2410_05265_amd.binding as b
    b.lib()
    return b


def inputs(M, K, step, seed):
    rng = np.random.default_rng(seed)
    x = (rng.standard_normal((M, K)) * 3 * step).astype(np.float16)
    ties = ((rng.integers(-10, 10, (M, K // 4)) + 0.5) * step).astype(np.float16)
    x[:, ::4] = np.nextafter(ties, (ties * rng.choice([0.5, 1, 2], ties.shape)).astype(np.float16))
    return x


def general(pq, call):
    prev = pq.pq_set_gemm_variant(2)          # the quantizer, then the tiled product
    try:
        return call()
    finally:
        pq.pq_set_gemm_variant(prev)


def bits(t):
    return host(t).view(np.uint16)


@pytest.mark.parametrize("step", [0.25, 0.3719])
@pytest.mark.parametrize("_,M,K,N", fused_shapes.ONE)
def test_one_matrix(pq, _, M, K, N, step):
    x = dev(inputs(M, K, step, M + K))
    w, sw = dev(synth.random_packed(N, K, seed=N + K, stream=7)), dev(synth.random_scales(N, seed=N))
    out, ws = pq.pq_linear(x, w, sw, step, 1)
    ref, wr = general(pq, lambda: pq.pq_linear(x, w, sw, step, 1))
    assert np.array_equal(host(ws)[: M * K // 2], host(wr)[: M * K // 2])
    assert np.array_equal(bits(out), bits(ref))


@pytest.mark.parametrize("_,M,K,Na,Nb", fused_shapes.TWO)
def test_two_matrices(pq, _, M, K, Na, Nb):
    step = 0.3719
    x = dev(inputs(M, K, step, M + K))
    wa, sa = dev(synth.random_packed(Na, K, seed=Na + K, stream=7)), dev(synth.random_scales(Na, seed=Na))
    wb, sb = dev(synth.random_packed(Nb, K, seed=Nb + K, stream=8)), dev(synth.random_scales(Nb, seed=Nb + 1))
    oa, ob, ws = pq.pq_linear2(x, wa, sa, wb, sb, step, 1)
    ra, rb, wr = general(pq, lambda: pq.pq_linear2(x, wa, sa, wb, sb, step, 1))
    assert np.array_equal(host(ws)[: M * K // 2], host(wr)[: M * K // 2])
    assert np.array_equal(bits(oa), bits(ra)) and np.array_equal(bits(ob), bits(rb))


@pytest.mark.parametrize("step", [0.25, 2.0 ** -20, 3.1e4])
def test_values_at_the_ends(pq, step):
    M, K, N = 8, 4096, 256
    x = inputs(M, K, np.float32(1.0), 3)
    x[0, :16] = [np.inf, -np.inf, np.nan, 0.0, -0.0, 6e-8, -6e-8, 65504, -65504, 1, -1, 6.1e-5, 0.125, -0.125, 1.875, -2.125]
    x[1] = np.nan
    x[2] = 0
    x[3] = np.inf
    w, sw = dev(synth.random_packed(N, K, seed=1, stream=7)), dev(synth.random_scales(N, seed=2))
    out, ws = pq.pq_linear(dev(x), w, sw, step, 0)
    ref, wr = general(pq, lambda: pq.pq_linear(dev(x), w, sw, step, 0))
    assert np.array_equal(host(ws)[: M * K // 2], host(wr)[: M * K // 2])
    assert np.array_equal(bits(out), bits(ref))


@pytest.mark.parametrize("M,K,N", [(5, 1024, 528), (16, 4096, 512)])
def test_against_the_oracle(pq, M, K, N):
    x, sx = synth.activations(M, K), O.calibrate_absmax(synth.calibration(K), 1)
    wq, sw = O.weight_rtn(synth.weights(N, K))
    w = O.pack(wq)
    out, ws = pq.pq_linear(dev(x), dev(w), dev(sw), float(sx), 1)
    codes = host(ws)[: M * K // 2].reshape(M, K // 2)
    assert np.array_equal(codes, O.linear(x, w, sw, sx, 1, return_all=True)["xq"])
    check_end_to_end(x, w, sw, sx, 1, host(out), codes)


@pytest.mark.parametrize("M,K", [(1, 4096), (4, 4096), (5, 4096), (16, 4096), (8, 2048)])
def test_output_over_the_tokens(pq, M, K):
    """In place: the codes are complete before any output is stored."""
    step, x = 0.3719, dev(inputs(M, K, 0.3719, M))
    w, sw = dev(synth.random_packed(K, K, seed=K, stream=7)), dev(synth.random_scales(K, seed=K))
    want, _ = pq.pq_linear(x, w, sw, step, 1)
    for second in (False, True):
        y, other = x.clone(), torch.empty_like(x)
        ws = torch.empty(1 << 16, dtype=torch.uint8, device="cuda")
        if second:
            pq.pq_linear2(y, w, sw, w, sw, step, 1, out_a=other, out_b=y, workspace=ws)
            assert np.array_equal(bits(other), bits(want))
        else:
            pq.pq_linear(y, w, sw, step, 1, out=y, workspace=ws)
        assert np.array_equal(bits(y), bits(want))


@pytest.mark.parametrize("M,K,N", [(1, 32, 16), (1, 32768, 528), (2, 544, 272), (3, 10912, 48), (4, 8192, 4112), (4, 8224, 48)])
def test_up_to_four_tokens(pq, M, K, N):
    """The fused launch of few tokens, with rows that the registers hold to the last piece, and more than that."""
    step, x = 0.3719, dev(inputs(M, K, 0.3719, M + K))
    w, sw = dev(synth.random_packed(N, K, seed=N + K, stream=7)), dev(synth.random_scales(N, seed=N))
    prev = pq.pq_set_gemm_variant(4)
    try:
        out, ws = pq.pq_linear(x, w, sw, step, 1)
        oa, ob, _ = pq.pq_linear2(x, w, sw, w[:16], sw[:16], step, 1)
    finally:
        pq.pq_set_gemm_variant(prev)
    ref, wr = general(pq, lambda: pq.pq_linear(x, w, sw, step, 1))
    assert np.array_equal(host(ws)[: M * K // 2], host(wr)[: M * K // 2])
    assert np.array_equal(bits(out), bits(ref)) and np.array_equal(bits(oa), bits(ref)) and np.array_equal(bits(ob), bits(ref)[:, :16])
