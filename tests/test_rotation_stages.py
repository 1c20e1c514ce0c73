"""The butterfly stages between lanes, written out in assembly: their wait states in the compiled kernels (CPU), and on the GPU
the rotation of rows whose result is known in closed form, for every block size, so that a wrong partner or sign shows."""

import os
import re
import subprocess

import numpy as np
import pytest

from paper_2410_05265_amd import build


@pytest.mark.parametrize("name", ["pq_rotate_quant.hip", "pq_gemm_f6.hip", "pq_decode.hip"])
def test_no_exchange_follows_its_writer_too_closely(name, tmp_path):
    """Between a vector instruction that writes a register and one that reads it through an exchange of lanes lie two others (or s_nop
    for them), along every straight run of the code and across labels."""
    out = str(tmp_path / "k.s")
    subprocess.run([build.HIPCC, *build.FLAGS, "-S", "--cuda-device-only", os.path.join(build.CSRC, name), "-o", out], check=True,
                   stderr=subprocess.DEVNULL)
    recent, seen = [], 0                                                 # (registers written, wait states since)
    for line in open(out):
        line = line.split(";")[0].strip()
        if not line or line.startswith(".") and not line.endswith(":") or line.endswith(":"):
            continue
        op, _, rest = line.partition(" ")
        if "_dpp" in op:
            seen += 1
            src = re.findall(r"v\d+", rest)[1]
            assert all(src not in regs for regs, age in recent if age < 2), line
        step = 1
        if op == "s_nop":
            step = int(rest, 0) + 1
        recent = [(regs, age + step) for regs, age in recent if age + step < 2]
        if op.startswith("v_") and not op.startswith("v_cmp"):
            m = re.match(r"v(\d+)\b|v\[(\d+):(\d+)\]", rest.strip())
            if m:
                lo, hi = (int(m.group(1)),) * 2 if m.group(1) else (int(m.group(2)), int(m.group(3)))
                recent.append(({"v%d" % r for r in range(lo, hi + 1)}, 0))
    assert seen > 50


@pytest.mark.gpu
@pytest.mark.parametrize("h", [2, 4, 8, 16, 32, 64, 128, 256, 512, 1024, 2048, 4096, 8192, 16384])
def test_unit_rows(h):
    """Row m has a single channel i of one block: its rotation is +-x / sqrt(h) with the sign of the parity of i & j at channel j.  x
    makes that 4 (or 60 at 8 bits) steps, so codes and per-token steps are exact."""
    import paper_2410_05265_amd.binding as pq
    import torch
    rng = np.random.default_rng(h)
    M, K = 37, 16384 if h > 4096 else 8192
    at = rng.integers(0, K, M)
    at[:4] = [0, h - 1, K - h, K - 1]
    sign = rng.choice([-1.0, 1.0], M)
    x = np.zeros((M, K), np.float16)
    x[np.arange(M), at] = (8.0 * sign).astype(np.float16)
    j, block = np.arange(K) % h, np.arange(K) // h
    parity = np.array([[bin(int(a)).count("1") & 1 for a in (j & (i % h))] for i in at])
    y = np.where(block[None] == (at // h)[:, None], np.where(parity == 1, -1, 1) * sign[:, None], 0)
    dx, value = torch.from_numpy(x).cuda(), 8.0 / np.sqrt(h)
    from oracle import unpack
    codes = pq.pq_rotate_quant(dx, h, float(value / 4))
    assert np.array_equal(unpack(codes.cpu().numpy()), 4 * y)
    codes, steps = pq.pq_rotate_quant_dynamic(dx, h, 1.0, 4)
    assert np.array_equal(unpack(codes.cpu().numpy()), 7 * y)
    assert np.allclose(steps.cpu().numpy(), value / 7, rtol=1e-6)
    out = pq.pq_rotate_quant8(dx, h, float(value / 60)).cpu().numpy().reshape(M, K // 32, 2, 16)
    assert np.array_equal(out.transpose(0, 1, 3, 2).reshape(M, K), 60 * y)
    zero = torch.zeros((3, K), dtype=torch.float16, device="cuda")
    assert not pq.pq_rotate_f16(zero, h).view(torch.int16).any()            # (+0 everywhere)
    assert np.allclose(pq.pq_rotate_f16(dx, h).cpu().numpy().astype(np.float64), y * value, rtol=1e-3)
