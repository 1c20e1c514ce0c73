"""Which launches a call makes, on the CPU (launch_log.py)."""

import os

import pytest

from launch_log import kernels, launches

pytestmark = pytest.mark.skipif(not os.path.exists("/opt/rocm/include/hip/hip_runtime_api.h"), reason="no HIP headers")

# calls that fuse quantizer and product when the output lies elsewhere
FUSED = [dict(fn="linear", M=M, K=K, N=K) for M, K in ((1, 4096), (4, 4096), (5, 4096), (16, 4096), (8, 2048))]
FUSED += [dict(fn="linear2", M=M, K=K, N=K) for M, K in ((1, 4096), (2, 4096), (3, 12288), (16, 8192))]
FUSED += [dict(fn="linear", M=2, K=4096, N=4096, h=128, variant=4), dict(fn="linear2", M=4, K=4096, N=4096, variant=4)]


@pytest.mark.parametrize("call", FUSED, ids=str)
def test_output_over_the_tokens_keeps_the_launches_apart(call):
    alone, *over = launches([call] + [dict(call, over=o) for o in ("out", "out_b")[:1 + (call["fn"] == "linear2")]])
    assert alone[0] == 0 and len(kernels(alone[1])) == 1
    for rc, events in over:
        first, *products = kernels(events)
        assert rc == 0 and first.startswith(("k_rotate_quant<", "k_rotate128")) and products
        assert not any(k.startswith(("k_rotate", "k_stream_fused")) for k in products)
