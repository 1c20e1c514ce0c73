"""The 4096-point rotation where its launches change shape: rows of the prepacked layer in groups of four and singly (all of
up to 768 blocks of 4096 channels, up to 256 behind the last 1024), rows of nibbles always singly; and the per-token quantizer of one to four
blocks a row, which rotates the same way.

A row's codes may depend on nothing but the row, so a long input repeats a few rows in an order of its own, and every copy
has to equal the codes of a call of those few rows (which the oracle checks), byte for byte."""

import numpy as np
import pytest
import torch

import oracle as O
from paper_2410_05265_amd import synth
from pq_testlib import dev, host
from test_gpu_gemm_f6 import tiles_by_definition

pytestmark = pytest.mark.gpu
H = 4096


@pytest.fixture(scope="module")
def pq():
    import paper_2410_05265_amd.binding as b
    b.lib()
    return b


@pytest.mark.parametrize("M,K", [(1, 4096), (31, 8192), (511, 4096), (513, 4096), (544, 8192), (991, 4096), (1023, 4096), (1025, 4096),
                                 (1279, 4096), (1281, 4096), (2300, 4096), (630, 8192), (383, 12288), (160, 28672)])
def test_rows_of_every_group_have_their_codes(pq, M, K):
    few = synth.activations(48, K, seed=K)
    order = np.random.default_rng(M).integers(0, 48, size=M)
    y = O.rotate(few, H)
    sx = np.float32(np.abs(y).max() / 7.0)
    part = O.unpack(host(pq.pq_rotate_quant(dev(few), H, float(sx)))).astype(np.int32)
    diff = part - O.quantize(y, sx).astype(np.int32)
    at = np.nonzero(diff)
    assert at[0].size <= 1e-3 * diff.size and np.all(np.abs(diff[at]) == 1)      # ties only
    x = torch.from_numpy(few).cuda()[torch.from_numpy(order).cuda()].contiguous()
    codes = host(pq.pq_rotate_quant(x, H, float(sx)))
    assert np.array_equal(O.unpack(codes), part[order])
    ws = torch.full((pq.pq_linear_f6_workspace_bytes(M, K, H),), 0x77, dtype=torch.uint8, device="cuda")
    w6 = pq.pq_repack_f6(dev(synth.random_packed(16, K, seed=1, stream=7)))
    pq.pq_linear_f6(x, w6, dev(synth.random_scales(16)), float(sx), H, workspace=ws)
    tiles = pq.pq_f6_tiles_bytes(M, K)
    assert np.array_equal(host(ws)[:tiles], tiles_by_definition(part[order]))
    off = (tiles + 255) // 256 * 256
    assert np.array_equal(host(ws)[off:off + M * K // 2].reshape(M, K // 2), codes)


@pytest.mark.parametrize("M,K", [(1, 4096), (3, 8192), (5, 12288), (70, 16384), (2, 20480)])
def test_dynamic_steps_and_codes_of_4096_point_blocks(pq, M, K):
    """(20480: past the longest row of that kernel, with the butterflies.)  The row maximum is a sum of 4096 terms in fp32:
    within a few ulps of the oracle's; codes against those of the oracle differ only at ties."""
    x = synth.activations(M, K, seed=M)
    if M > 2:
        x[1] = 0                                                    # step 1, codes 0
        x[2, :K - H] = 0                                            # the maximum in the last block
    y = O.rotate(x, H)
    want_q, want_s = O.quantize_dynamic(y, 0.875, 4)
    q, s = pq.pq_rotate_quant_dynamic(dev(x), H, 0.875, 4)
    s, got = host(s), O.unpack(host(q)).astype(np.int32)
    assert np.all(np.abs(s.view(np.int32).astype(np.int64) - np.asarray(want_s, np.float32).view(np.int32)) <= 8)
    diff = got - want_q.astype(np.int32)
    at = np.nonzero(diff)
    assert at[0].size <= 1e-3 * diff.size and np.all(np.abs(diff[at]) == 1)
    if M > 2:
        assert s[1] == 1.0 and not got[1].any() and not got[2, :K - H].any()


def test_dynamic_rows_past_the_threads_of_one_launch(pq):
    """2^22 rows of 16384 channels are 2^32 threads, one launch's limit (137 GB of input; the last rows and the ones around the
    borders of the launches are looked at)."""
    M, K = (1 << 22) + 3, 16384
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < M * K * 5 // 2 + (8 << 30):
        pytest.skip("needs 172 GB of free device memory")
    few = synth.activations(8, K, seed=22)
    part, steps = pq.pq_rotate_quant_dynamic(dev(few), H, 0.875, 4)
    x = torch.empty((M, K), dtype=torch.float16, device="cuda")
    at = torch.tensor([0, (1 << 20) - 1, 1 << 20, (1 << 21) + 1, 3 << 20, (1 << 22) - 1, 1 << 22, M - 1], device="cuda")
    for i, row in enumerate(at.tolist()):
        x[row] = torch.from_numpy(few[i])
    codes, got = pq.pq_rotate_quant_dynamic(x, H, 0.875, 4)
    assert torch.equal(codes[at], part) and torch.equal(got[at], steps)
    del x, codes
    torch.cuda.empty_cache()
