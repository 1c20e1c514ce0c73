"""The butterfly stages between lanes, written out in assembly: their wait states in the compiled kernels (CPU), and on the GPU
the rotation of rows whose result is known in closed form, for every block size, so that a wrong partner or sign shows."""

import os
import re
import subprocess

import numpy as np
import pytest

from paper_2410_05265_amd import build
from test_matrix_wait_states import NO_RESULT, functions, registers, violations


# every source that the rotation is compiled into
SOURCES = [os.path.basename(f) for f in build.sources() if '#include "pq_rotate.h"' in open(f).read()]
# states between a vector instruction that writes a register, or the lanes' mask, and an exchange of lanes that reads it; between a matrix
# instruction and an exchange in the stages' assembly (the compiler sees to its own)
AFTER_WRITE, AFTER_MASK, AFTER_MATRIX = 2, 5, 18
EXCHANGE = ("_dpp", "v_permlane16_swap", "v_permlane32_swap")


def step(pending, ins, report):
    """As its namesake of the matrix instructions: pending maps (register or "mask") to the states that still have to pass."""
    op, _, rest = ins.line.partition(" ")
    operands = [registers(o) for o in re.split(r",(?![^\[]*\])", rest)] if rest else []
    if any(e in op for e in EXCHANGE):
        reads = operands[0] | operands[1] if "swap" in op else operands[1]
        for key in reads | {"mask"} | {("matrix", reg) for reg in reads if ins.in_asm}:
            if key in pending:
                report.append("%s: %s %d states too early" % (ins.line, key, pending[key]))
    pending = {k: left - ins.states for k, left in pending.items() if left > ins.states}
    if op.startswith("v_cmpx"):
        pending["mask"] = AFTER_MASK
    elif op.startswith("v_") and not op.startswith(NO_RESULT) and operands:
        for reg in operands[0] | (operands[1] if "swap" in op else frozenset()):
            if op.startswith("v_mfma"):
                pending["matrix", reg] = AFTER_MATRIX
            else:
                pending[reg] = AFTER_WRITE
                pending.pop(("matrix", reg), None)
    return pending


@pytest.fixture(scope="module")
def compiled(tmp_path_factory):
    if not os.path.exists(build.HIPCC):
        pytest.skip("hipcc not installed")
    folder = tmp_path_factory.mktemp("asm")
    procs = [(s, subprocess.Popen([build.HIPCC, *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, s), "-o", str(folder / s)],
                                  stderr=subprocess.PIPE, text=True)) for s in SOURCES]
    out = {}
    for s, pr in procs:
        _, err = pr.communicate()
        assert pr.returncode == 0, err[-4000:]
        out[s] = functions((folder / s).read_text())
    return out


def test_sources_are_found():
    assert {"pq_rotate_quant.hip", "pq_gemm_f6.hip", "pq_decode.hip", "pq_stream_mfma.hip", "pq_calibrate.hip"} <= set(SOURCES)


@pytest.mark.parametrize("name", SOURCES)
def test_no_exchange_follows_its_writer_too_closely(compiled, name):
    """Along every path through the compiled kernels: the compiler does not see into the stages' assembly, neither what they read nor that
    they write."""
    exchanges = 0
    for kernel, (blocks, labels) in compiled[name].items():
        exchanges += sum("_dpp" in i.line for b in blocks for i in b)
        bad = violations(blocks, labels, step)
        assert not bad, "%s: %d, first %s" % (kernel, len(bad), bad[:3])
    assert exchanges > 50


@pytest.mark.parametrize("lines,bad", [
    (["v_add_f32_e32 v1, v2, v3", "v_fmac_f32_dpp v1, v1, v4 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf bound_ctrl:1"], 1),
    (["v_add_f32_e32 v1, v2, v3", "s_nop 1", "v_fmac_f32_dpp v1, v1, v4 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf bound_ctrl:1"], 0),
    (["v_add_f32_e32 v1, v2, v3", "s_nop 0", "s_cbranch_scc1 .LBB0_1", "s_nop 7", ".LBB0_1:", "v_mov_b32_dpp v5, v1 row_half_mirror row_mask:0xf bank_mask:0xf bound_ctrl:1"], 0),
    (["v_add_f32_e32 v1, v2, v3", "s_cbranch_scc1 .LBB0_1", "s_nop 7", ".LBB0_1:", "v_mov_b32_dpp v5, v1 row_half_mirror row_mask:0xf bank_mask:0xf bound_ctrl:1"], 1),
    (["v_cmpx_lt_u32_e32 v1, v2", "s_nop 3", "v_mov_b32_dpp v5, v4 row_ror:8 row_mask:0xf bank_mask:0xf"], 1),
    (["v_mfma_f32_32x32x16_f16 v[0:15], v[16:19], v[20:23], v[0:15]", "s_nop 7", ";;#ASMSTART", "v_mov_b32_dpp v25, v3 row_ror:8 row_mask:0xf bank_mask:0xf"], 1),
    (["v_mov_b32_dpp v5, v4 row_ror:8 row_mask:0xf bank_mask:0xf", "v_permlane32_swap_b32_e32 v6, v5"], 1)])
def test_the_count_itself(lines, bad):
    blocks, labels = functions("_Zk:\n%s\ts_endpgm\n.Lfunc_end0:\n" % "".join(t + "\n" if t.endswith((":", "START")) else "\t%s\n" % t for t in lines))["_Zk"]
    assert (len(violations(blocks, labels, step)) > 0) == bool(bad)


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
