"""What library calls would launch, read without a GPU: the calls run in a process of their own on a stand-in for the runtime's
launch entries (launch_log.cpp).  `launches(calls)`: one entry per call, its status and its ("launch" or "allow", kernel, workgroups,
bytes of dynamic LDS) in order.  A call is a dict: fn ("linear", "linear2", "gemm": the product of
packed codes, "f6": of prepacked ones, "f6_two": the layer of two prepacked matrices), M, K, N (N2: of the second matrix), h, variant
(pq_set_gemm_variant), over ("out": the output lies over the tokens, "out_b": the second one does), start (bytes that the outputs start behind a line)."""

import ctypes
import functools
import json
import os
import re
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_2410_05265_amd", "libpq.so")


@functools.lru_cache(None)
def _stand_in():
    out = os.path.join(tempfile.mkdtemp(prefix="pq_launch_log"), "launch_log.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__=1", "-I/opt/rocm/include",
                    os.path.join(HERE, "launch_log.cpp"), "-o", out], check=True)
    return out


def launches(calls):
    r = subprocess.run([sys.executable, os.path.abspath(__file__), _stand_in(), LIB], input=json.dumps(calls), capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-4000:]
    return [(rc, [tuple(e) for e in events]) for rc, events in json.loads(r.stdout)]


def kernels(events):
    return [e[1] for e in events if e[0] == "launch"]


def _main():
    log = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
    log.launch_log.restype = ctypes.c_char_p
    pq = ctypes.CDLL(sys.argv[2])
    i32, i64, f32, p, size = ctypes.c_int32, ctypes.c_int64, ctypes.c_float, ctypes.c_void_p, ctypes.c_size_t
    x, wa, wb, sa, sb, oa, ob, ws = (p((i + 1) << 40) for i in range(8))      # (far apart and never read)
    out = []
    for c in json.load(sys.stdin):
        M, K, N, N2, h, room = i64(c["M"]), i64(c["K"]), i64(c["N"]), i64(c.get("N2", c["N"])), i32(c.get("h", 1)), size(1 << 36)
        over = c.get("over")
        a, b = (x if over == o else p(t.value + c.get("start", 0)) for o, t in (("out", oa), ("out_b", ob)))
        pq.pq_set_gemm_variant(c.get("variant", 0))
        log.launch_log_clear()
        fn = c["fn"]
        if fn == "linear":
            rc = pq.pq_linear(x, wa, sa, f32(0.5), h, M, N, K, a, ws, room, p(0))
        elif fn == "linear2":
            rc = pq.pq_linear2(x, wa, sa, N, a, wb, sb, N2, b, f32(0.5), h, M, K, ws, room, p(0))
        elif fn == "gemm":
            rc = pq.pq_w4a4_gemm(x, wa, sa, f32(0.5), M, N, K, a, p(0), p(0))
        elif fn == "f6":
            rc = pq.pq_w4a4_gemm_f6(x, wa, sa, f32(0.5), M, N, K, a, p(0), p(0))
        else:
            rc = pq.pq_linear2_f6(x, wa, sa, N, a, wb, sb, N2, b, f32(0.5), h, M, K, ws, room, p(0))
        events = []
        for line in log.launch_log().decode().splitlines():
            what, name, grid, lds = line.split("\t")
            events.append((what, re.search(r"(k_\w+(?:<[^(]*>)?)", name).group(1), int(grid), int(lds)))
        out.append((rc, events))
    json.dump(out, sys.stdout)


if __name__ == "__main__":
    _main()
