"""Rotations on the matrix pipe: a token has the same codes in every call, form and batch (blocks of 4096 channels), and
the quantizer with a zero-point of 8 is the symmetric one.

The inputs are made so that sums taken in another order give other codes: half of the channels hold one large value with
the signs of a Hadamard row (every output but one cancels it), the others hold small ones, so the fp32 rounding of the
large partial sums reaches the small outputs.  Each test checks on the CPU that its inputs do tell orders apart."""

import numpy as np
import pytest

import oracle as O
from paper_2410_05265_amd import synth
from pq_testlib import dev, host

pytestmark = pytest.mark.gpu
H = 4096


@pytest.fixture(scope="module")
def pq():
    import paper_2410_05265_amd.binding as b
    b.lib()
    return b


def order_sensitive(rows, K, seed, h=H):
    rng = np.random.default_rng(seed)
    x = rng.normal(0.0, 0.06, size=(rows, K // h, h)).astype(np.float16)
    sign = np.array([bin(i & 1234).count("1") & 1 for i in range(h)])
    x[:, :, 0::2] = np.where(sign[0::2], -2000.0, 2000.0).astype(np.float16)
    return x.reshape(rows, K), np.float32(1.2 / 64)


def butterfly_codes(x, sx, h=H):
    """The codes of plain fp32 butterflies, one of the other orders."""
    v = x.astype(np.float32).reshape(-1, h)
    d = 1
    while d < h:
        v = v.reshape(-1, h // (2 * d), 2, d)
        v = np.stack([v[:, :, 0] + v[:, :, 1], v[:, :, 0] - v[:, :, 1]], axis=2).reshape(-1, h)
        d *= 2
    return np.clip(np.rint(v * np.float32(1.0 / (np.float64(sx) * np.sqrt(h)))), -8, 7).astype(np.int8).reshape(x.shape)


# tokens of a call, channels, kernel variant: the shapes whose automatic choice is the fused launch (1 x 4096 .. 1 x 16384,
# 2 x 4096; one and two weight rows per wavefront), and those that only the forced one takes
@pytest.mark.parametrize("M,K,N,variant", [(1, 4096, 64, 0), (2, 4096, 64, 0), (1, 8192, 64, 0), (1, 16384, 64, 0), (1, 4096, 8208, 0),
                                           (3, 4096, 64, 0), (3, 8192, 64, 4), (4, 12288, 64, 4)])
def test_few_tokens_have_the_codes_of_a_batch(pq, M, K, N, variant):
    rows = 12
    x, sx = order_sensitive(rows, K, seed=M + K)
    batch = host(pq.pq_rotate_quant(dev(x), H, float(sx)))
    assert (O.unpack(batch) != butterfly_codes(x, sx)).any()
    w, s = dev(synth.random_packed(N, K, seed=N, stream=7)), dev(synth.random_scales(N, seed=N))
    w6 = pq.pq_repack_f6(w)
    for r in range(0, rows, M):
        part = dev(x[r:r + M])
        f6, _ = pq.pq_linear_f6(part, w6, s, float(sx), H)
        prev = pq.pq_set_gemm_variant(variant)
        try:
            out, ws = pq.pq_linear(part, w, s, float(sx), H)
            a, b, ws2 = pq.pq_linear2(part, w, s, w, s, float(sx), H)
        finally:
            pq.pq_set_gemm_variant(prev)
        for codes in (ws, ws2):
            assert np.array_equal(host(codes)[: M * K // 2].reshape(M, K // 2), batch[r:r + M])
        for got in (f6, a, b):
            assert np.array_equal(host(got).view(np.uint16), host(out).view(np.uint16))


@pytest.mark.parametrize("M,K,h", [(70, 4096, 4096), (3, 8192, 4096), (600, 1152, 128)])
def test_zero_point_eight_is_the_symmetric_quantizer(pq, M, K, h):
    """Also for the blocks whose rotation runs on the matrix pipe."""
    x, sx = order_sensitive(M, K, seed=M + K, h=h)
    codes = host(pq.pq_rotate_quant(dev(x), h, float(sx)))
    assert (O.unpack(codes) != butterfly_codes(x, sx, h)).any()
    assert np.array_equal(host(pq.pq_rotate_quant_zp(dev(x), h, float(sx), 8)), codes)


def test_one_hot_and_constant_rows(pq):
    """Rows whose rotation is known in closed form.  A one-hot row of 3 becomes +-3 / 64 in its block, the signs a row of the
    Hadamard matrix: codes +-7 there and 0 in the other blocks.  A constant row of 0.25 becomes 16 in the first channel of
    every block."""
    K, w = 3 * H, synth.random_packed(16, 3 * H, seed=1, stream=7)
    at = [1 << b for b in range(12)] + [(77 * r + 13) % H for r in range(58)]          # every bit alone, then mixtures
    x = np.zeros((len(at), K), dtype=np.float16)
    want = np.zeros((len(at), K), dtype=np.int8)
    j = np.arange(H)
    for r, i in enumerate(at):
        block = r % 3
        x[r, block * H + i] = np.float16(3.0)
        parity = np.array([bin(i & c).count("1") & 1 for c in j])
        want[r, block * H:(block + 1) * H] = 7 - 14 * parity
    sx = 3.0 / 64 / 7
    assert np.array_equal(O.unpack(host(pq.pq_rotate_quant(dev(x), H, sx))), want)
    dw, s = dev(w), dev(synth.random_scales(16))
    _, ws = pq.pq_linear_f6(dev(x), pq.pq_repack_f6(dw), s, sx, H)
    codes = host(ws)[(pq.pq_f6_tiles_bytes(len(at), K) + 255) // 256 * 256:][:len(at) * K // 2].reshape(len(at), K // 2)
    assert np.array_equal(O.unpack(codes), want)
    for r in (0, 1, 11, 12, 69):                                                       # the fused launch of one token
        _, ws = pq.pq_linear(dev(x[r:r + 1]), dw, s, sx, H)
        assert np.array_equal(O.unpack(host(ws)[:K // 2].reshape(1, K // 2)), want[r:r + 1])
    const = np.full((5, K), 0.25, dtype=np.float16)
    got = O.unpack(host(pq.pq_rotate_quant(dev(const), H, 16.0 / 7)))
    assert (got[:, ::H] == 7).all() and np.count_nonzero(got) == 5 * 3
