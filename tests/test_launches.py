"""Which launches a call makes, on the CPU (launch_log.py)."""

import os

import pytest

import fused_shapes
from launch_log import kernels, launches
from packed_tiles import TILES
from square_tiles import LARGE, ONE, STREAM_ONE, STREAM_TWO, TWO

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


def allowed_before_launched(events):
    """Kernels launched with more than 64 KiB of dynamic LDS and not allowed as much before."""
    limit, late = {}, []
    for what, kernel, _, lds in events:
        if what == "allow":
            limit[kernel] = lds
        elif lds > 65536 and limit.get(kernel, 0) < lds:
            late.append(kernel)
    return late


def test_every_kernel_is_allowed_its_dynamic_lds():
    """The runtime is told per kernel.  One process, as a program's: what one kernel was told must not count for another."""
    calls = [dict(fn="linear", M=M, K=K, N=N, variant=v) for v in (0, 1, 2, 4, 5) for M in (1, 3, 5, 8, 13, 16, 24, 40, 96, 300, 777, 2048)
             for K, N in ((256, 16), (1024, 4096), (4096, 528), (4096, 14336), (8192, 8192), (14336, 4096), (8192, 528), (65536, 16))]
    calls += [dict(fn="linear2", M=M, K=K, N=N) for M in (2, 4, 9, 16, 100) for K, N in ((1024, 272), (8192, 528), (8192, 11008), (12288, 14336))]
    calls += [dict(fn=f, M=M, K=K, N=N) for f in ("f6", "f6_two") for M in (40, 333, 700, 1111, 2048, 5000) for K in (1024, 4096, 11008)
              for N in (1024, 4096, 12288, 28672)]
    done = launches(calls)
    events = [e for rc, ev in done if rc == 0 for e in ev]
    used = {e[1] for e in events if e[0] == "launch"}
    assert not allowed_before_launched(events)
    for family, count in (("k_stream_fused<", 4), ("k_stream_mfma<4", 3), ("k_gemm_f6_square<", 10), ("k_decode<", 6)):
        assert sum(k.startswith(family) for k in used) >= count, (family, used)


@pytest.mark.parametrize("cases,fn,streamed", [(ONE, "f6", 0), (TWO, "f6_two", 0), (STREAM_ONE, "f6", 1), (STREAM_TWO, "f6_two", 1), (LARGE, "f6", 0)])
def test_near_square_tiles_and_how_they_store(cases, fn, streamed):
    done = launches([dict(fn=fn, M=M, K=K, N=N) for _, M, N, K in cases])
    want = ["k_gemm_f6_square<%d, %d, %s, %s>" % (t // 10, t % 10, ("false", "true")[fn == "f6_two"], ("false", "true")[streamed])
            for t, _, _, _ in cases]
    assert [kernels(events)[-1] for _, events in done] == want


@pytest.mark.parametrize("fn,M,K,N", [("f6", 2319, 1024, 10048), ("f6_two", 772, 1024, 9920)])
def test_outputs_that_start_within_a_line(fn, M, K, N):
    """The start of the output counts as the length of its rows does: whole lines from 128 bytes on, halves from 64."""
    done = launches([dict(fn=fn, M=M, K=K, N=N, start=s) for s in (0, 128, 64, 32, 16)])
    assert [kernels(events)[-1].endswith("true>") for _, events in done] == [True, True, True, False, False]


# channels in under 6144: tokens, channels in, channels out; measured us of the other kernel and of near-square tiles, three sets of operands
@pytest.mark.parametrize("fn,M,K,N,other_us,square_us", [
    ("f6_two", 1024, 4096, 22016, 129.5, 108.2), ("f6_two", 2048, 4096, 22016, 236.5, 212.0), ("f6_two", 3000, 4096, 22016, 364.4, 347.4),
    ("f6_two", 4889, 1280, 6496, 77.3, 81.4), ("f6_two", 1979, 1280, 8800, 45.8, 47.6), ("f6", 2048, 4096, 14336, 66.7, 67.6),
    ("f6", 4096, 3072, 16384, 126.8, 119.3), ("f6", 4096, 3072, 32768, 253.9, 249.9), ("f6", 4096, 3072, 65536, 550.8, 571.3),
    ("f6", 8192, 4096, 16384, 301.4, 285.6), ("f6", 3403, 3840, 14976, 121.4, 125.9), ("f6", 1004, 2816, 22672, 47.1, 51.6),
    ("f6", 641, 3072, 17920, 28.2, 25.3), ("f6", 1505, 4864, 22784, 102.1, 94.3), ("f6", 5024, 1280, 17344, 110.8, 97.2)])
def test_near_square_tiles_of_short_rows_where_they_were_measured_faster(fn, M, K, N, other_us, square_us):
    (_, events), = launches([dict(fn=fn, M=M, K=K, N=N)])
    assert kernels(events)[-1].startswith("k_gemm_f6_square<") == (square_us < other_us)


def test_unrotated_tokens_have_a_kernel_of_their_own_up_to_what_registers_hold():
    calls = [dict(fn="linear", M=M, K=K, N=528, h=h, variant=4) for M, K, h in ((1, 32768, 1), (4, 8192, 0), (4, 8224, 1), (1, 32768, 64), (1, 4096, 4096))]
    modes = [kernels(events)[0].split(", ")[3] for _, events in launches(calls)]
    assert modes == ["3", "3", "1", "1", "2"]


@pytest.mark.parametrize("cases", [fused_shapes.ONE, fused_shapes.TWO])
def test_fused_launch_of_up_to_16_tokens(cases):
    done = launches([dict(fn="linear2" if len(c) == 5 else "linear", M=c[1], K=c[2], N=c[3], N2=c[-1]) for c in cases])
    assert [kernels(events) for _, events in done] == [["k_stream_fused<%d, %d>" % c[0]] for c in cases]


def test_every_fused_kernel_runs_several_tasks_of_several_units():
    """What the shapes above are there for: each kernel, and with more than one unit a wavefront also several tasks a workgroup, so that tasks end
    inside a round and sums leave before the last one."""
    seen = set()
    for c in fused_shapes.ONE + fused_shapes.TWO:
        P, N = c[2] // 256, sum(c[3:])
        slices = 16 if P > 8 else (8 if P > 4 else 4)
        units, tasks = -(-P // slices), -(-(N // 16) // (16 // slices))
        seen.add((c[0], "units" if units > 1 else "unit", "tasks" if -(-tasks // min(tasks, 256)) > 2 else "task"))
    assert {k for k, _, _ in seen} == {(2, 8), (4, 8), (2, 16), (4, 16)}
    assert {((4, 8), "units", "tasks"), ((4, 16), "units", "tasks"), ((4, 8), "unit", "tasks")} <= seen


def test_every_packed_tile_has_its_shape():
    done = launches([dict(fn="gemm", M=M, K=K, N=N, variant=2) for _, M, N, K in TILES])
    assert [kernels(events)[0].startswith("k_gemm_dma<%d, %d," % (t // 1000, t % 1000)) for (t, _, _, _), (_, events) in zip(TILES, done)] == [True] * 13


# tokens, channels in, channels out; measured us of the small tiles and of the tiled kernel
@pytest.mark.parametrize("M,K,N,small_us,tiled_us", [
    (137, 6656, 22080, 41.6, 32.9), (181, 6656, 24560, 43.8, 33.4), (143, 7680, 23120, 46.5, 36.2), (588, 12672, 7072, 68.9, 57.0),
    (546, 9216, 7632, 50.7, 44.3), (342, 18560, 11008, 93.9, 86.1), (183, 6016, 5696, 14.9, 18.7), (292, 19456, 4992, 43.1, 52.5),
    (225, 17920, 6704, 41.5, 49.9), (668, 7936, 2384, 22.9, 25.4), (108, 21888, 15920, 69.6, 74.8), (200, 4096, 6144, 10.8, 13.9)])
def test_small_tiles_where_they_were_measured_faster(M, K, N, small_us, tiled_us):
    (_, events), = launches([dict(fn="gemm", M=M, K=K, N=N)])
    assert kernels(events)[0].startswith("k_gemm_i8_ksplit<") == (small_us < tiled_us)
