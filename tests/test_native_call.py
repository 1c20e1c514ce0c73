"""The native call path of pq_linear and pq_linear2: what it declines (the Python path then words the error), and on the GPU that it
passes on what the ctypes path does, on the current stream, from several threads."""

import os
import subprocess
import sys
import threading

import numpy as np
import pytest
import torch

import paper_2410_05265_amd.binding as b
from paper_2410_05265_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def tensors(device, M=3, K=512, N=64):
    g = torch.Generator().manual_seed(1)
    return [torch.randn((M, K), generator=g).half().to(device), torch.randint(0, 256, (N, K // 2), generator=g, dtype=torch.uint8).to(device),
            (torch.rand(N, generator=g) + 0.5).to(device)]


def test_declines_what_is_not_plain():
    b.lib()
    x, w, s = tensors("cpu")
    out, ws = torch.empty(3, 64).half(), torch.empty(4096, dtype=torch.uint8)
    assert b._call.linear(x, w, s, 0.5, 1, out, ws) == -1                     # not on the GPU
    assert b._call.linear(x, w, s, 0.5, 1, out) == -1 and b._call.linear() == -1
    assert b._call.linear(None, w, s, 0.5, 1, out, ws) == -1
    assert b._call.linear2(x, w, s, w, s, 0.5, 1, out, out, ws) == -1
    with pytest.raises(TypeError):
        b.pq_linear(x, w, s, 0.5, 1, out=out, workspace=ws)
    with pytest.raises(TypeError):
        b.pq_linear2(x, w, s, w, s, 0.5, 1, out_a=out, out_b=out, workspace=ws)


SCRIPT = """
import sys, warnings
from paper_2410_05265_amd import binding as b, build
%s
with warnings.catch_warnings(record=True) as w:
    warnings.simplefilter("always")
    assert b.lib().pq_version() >= 100 and b._call is b._Declines and b._call.linear(1) == b._call.linear2(1) == -1
    assert any("native call path" in str(x.message) for x in w)
import torch
x, k, s = torch.zeros(3, 512).half(), torch.zeros(64, 256, dtype=torch.uint8), torch.ones(64)
try:
    b.pq_linear(x, k, s, 0.5, 1, out=torch.empty(3, 64).half(), workspace=torch.empty(4096, dtype=torch.uint8))
except TypeError:
    print("declined by the Python path")
"""


@pytest.mark.parametrize("how", ["absent", "of another torch", "unreadable"])
def test_library_loads_without_the_native_call_path(how, tmp_path):
    broken = tmp_path / "broken.so"
    broken.write_bytes(b"not a library")
    setup = {"absent": "b.CALL_PATH = %r" % str(tmp_path / "none.so"), "unreadable": "b.CALL_PATH = %r" % str(broken),
             "of another torch": "import importlib, torch; torch.__version__ = '0.0'; importlib.reload(b); assert build._call_is_stale()"}[how]
    r = subprocess.run([sys.executable, "-c", SCRIPT % setup], cwd=ROOT, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and "declined by the Python path" in r.stdout, r.stderr[-2000:]


def test_build_goes_on_without_a_host_compiler(monkeypatch, capfd):
    monkeypatch.setenv("PATH", "/nonexistent")
    before = os.path.getmtime(b.CALL_PATH)
    assert not build._build_call() and "ctypes" in capfd.readouterr().err
    assert os.path.getmtime(b.CALL_PATH) == before and not build._call_is_stale()


def test_python_path_checks_the_callers_buffers(monkeypatch):
    """On the CPU, with the checks of the operands taken out of the way: the output's and the workspace's own checks."""
    b.lib()
    monkeypatch.setattr(b, "_dev", lambda *a: None)
    monkeypatch.setattr(torch.Tensor, "is_pinned", lambda t: True)
    launched = []
    monkeypatch.setattr(b, "lib", lambda: type("L", (), {"pq_linear": staticmethod(lambda *a: launched.append(a) or 0),
                                                         "pq_linear2": staticmethod(lambda *a: launched.append(a) or 0)}))
    monkeypatch.setattr(b, "_stream", lambda: 0)
    x, w, s = tensors("cpu")
    out, ws = torch.empty(3, 64).half(), torch.empty(4096, dtype=torch.uint8)
    for o, k in ((out[:2], ws), (out.float(), ws), (torch.empty(64, 3).half().t(), ws), (out, torch.empty(8192, dtype=torch.uint8)[::2])):
        with pytest.raises((TypeError, ValueError)):
            b.pq_linear(x, w, s, 0.5, 1, out=o, workspace=k)
        for oa, ob in ((o, out), (out, o)):
            with pytest.raises((TypeError, ValueError)):
                b.pq_linear2(x, w, s, w, s, 0.5, 1, out_a=oa, out_b=ob, workspace=k)
    assert not launched
    b.pq_linear(x, w, s, 0.5, 1, out=torch.empty(5, 64).half(), workspace=ws)
    assert len(launched) == 1


@pytest.mark.gpu
def test_same_refusals_as_the_python_path():
    b.lib()
    x, w, s = tensors("cuda")
    out, ws = torch.empty((3, 64), dtype=torch.float16, device="cuda"), torch.empty(4096, dtype=torch.uint8, device="cuda")

    class Sub(torch.Tensor):
        pass

    declined = [(x.t().contiguous().t(), w, s, 0.5, 1), (x.float(), w, s, 0.5, 1), (x, w.view(torch.int8), s, 0.5, 1), (x, w, s.double(), 0.5, 1),
                (x, w[:, :128].contiguous(), s, 0.5, 1), (x, w, s[:32].contiguous(), 0.5, 1), (x.view(3, 2, 256), w, s, 0.5, 1),
                (x, w, s, np.float32(0.5), 1), (x, w, s, 0.5, np.int64(1)), (x, w, s, 0.5, 1 << 40), (x.as_subclass(Sub), w, s, 0.5, 1)]
    for a in declined:
        assert b._call.linear(*a, out, ws) == -1
    for a in declined[:7]:
        with pytest.raises((TypeError, ValueError)):
            b.pq_linear(*a, out=out, workspace=ws)
    ref, _ = b.pq_linear(x, w, s, 0.5, 1)
    for a in declined[7:9] + declined[10:]:
        got, _ = b.pq_linear(*a, out=out.zero_(), workspace=ws)
        assert got is out and torch.equal(got, ref)
    for step, ws_, status in ((0.0, ws, b.PQ_ERR_SCALE), (0.5, ws[:256], b.PQ_ERR_WORKSPACE), (0.5, ws[1:], b.PQ_ERR_ALIGN)):
        with pytest.raises(b.PQError) as e:
            b.pq_linear(x, w, s, step, 1, out=out, workspace=ws_)
        assert e.value.status == status


@pytest.mark.gpu
def test_outputs_streams_and_threads():
    x, w, s = tensors("cuda", 5, 4096, 1040)
    ref, refws = b.pq_linear(x, w, s, 0.37, 1)
    ra, rb, _ = b.pq_linear2(x, w, s, w[:528], s[:528], 0.37, 1)
    torch.cuda.synchronize()
    errors = []

    def work(i):
        try:
            st = torch.cuda.Stream()
            with torch.cuda.stream(st):
                out, ws = torch.empty_like(ref), torch.empty(65536, dtype=torch.uint8, device="cuda")
                oa, ob = torch.empty_like(ra), torch.empty_like(rb)
                for _ in range(20):
                    o, k = b.pq_linear(x, w, s, 0.37, 1, out=out, workspace=ws)
                    codes = k[: 5 * 2048].clone()
                    b.pq_linear2(x, w, s, w[:528], s[:528], 0.37, 1, out_a=oa, out_b=ob, workspace=ws)
            st.synchronize()
            assert o is out and k is ws and torch.equal(out, ref) and torch.equal(codes, refws[: 5 * 2048])
            assert torch.equal(oa, ra) and torch.equal(ob, rb)
        except Exception as e:            # reported by the main thread
            errors.append(e)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    [t.start() for t in threads]
    [t.join() for t in threads]
    assert not errors


@pytest.mark.gpu
def test_runs_on_the_current_stream():
    x, w, s = tensors("cuda", 1, 4096, 4096)
    out, ws = torch.empty((1, 4096), dtype=torch.float16, device="cuda"), torch.empty(65536, dtype=torch.uint8, device="cuda")
    ref = b.pq_linear(x, w, s, 0.37, 1)[0].clone()
    b.pq_linear(x, w, s, 0.37, 1, out=out, workspace=ws)
    g = torch.cuda.CUDAGraph()
    out.zero_()
    with torch.cuda.graph(g):                  # a launch on any other stream than the capturing one would not be recorded
        b.pq_linear(x, w, s, 0.37, 1, out=out, workspace=ws)
    torch.cuda.synchronize()
    for _ in range(3):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref)

@pytest.mark.gpu
@pytest.mark.parametrize("two", [False, True])
def test_outputs_and_workspaces_that_kernels_must_not_write(two):
    """Too small, of another type, not contiguous, not on the GPU: refused before anything is launched, on either path; a larger
    output, a workspace of another type and pinned memory are accepted as before."""
    b.lib()
    x, w, s = tensors("cuda")
    M, N = 3, 64
    ws, good = torch.empty(4096, dtype=torch.uint8, device="cuda"), torch.empty((M, N), dtype=torch.float16, device="cuda")
    ref, _ = b.pq_linear(x, w, s, 0.5, 1)
    half = dict(dtype=torch.float16, device="cuda")

    def call(out, workspace, native):
        saved, b._call = b._call, b._call if native else b._Declines
        try:
            if two:
                b.pq_linear2(x, w, s, w, s, 0.5, 1, out_a=out, out_b=good, workspace=workspace)
                b.pq_linear2(x, w, s, w, s, 0.5, 1, out_a=good, out_b=out, workspace=workspace)
            else:
                b.pq_linear(x, w, s, 0.5, 1, out=out, workspace=workspace)
        finally:
            b._call = saved

    bad = [(torch.empty((M - 1, N), **half), ws), (torch.empty((M, N), device="cuda"), ws), (torch.empty((N, M), **half).t(), ws),
           (torch.empty((M, 2 * N), **half)[:, ::2], ws), (torch.empty((M, N), dtype=torch.float16), ws),
           (good, torch.empty(8192, dtype=torch.uint8, device="cuda")[::2]), (good, torch.empty(4096, dtype=torch.uint8))]
    for native in (True, False):
        for out, workspace in bad:
            with pytest.raises((TypeError, ValueError)):
                call(out, workspace, native)
        for out, workspace in ((torch.zeros((M + 2, N), **half), ws), (torch.zeros(M * N, **half), torch.empty(4096, device="cuda")),
                               (torch.zeros((M, N), dtype=torch.float16).pin_memory(), ws)):
            call(out, workspace, native)
            torch.cuda.synchronize()
            assert torch.equal(out.reshape(-1)[:M * N].cuda(), ref.reshape(-1))

