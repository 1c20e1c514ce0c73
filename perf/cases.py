"""The work whose time counts: calls of the layer as an inference program makes them.

A case is one call (or one producer and one product) through the Python binding, with the weights quantized, packed
and, on the prepacked path, repacked beforehand, and with output and workspace buffers that the program keeps.
Sizes are the linears of the Llama-2-7B, Llama-3-8B and Llama-3-70B blocks and generic ones between them; token counts
run from one decoded token to a prefill of some thousands.  Activations and weights follow the recipe of
`paper_2410_05265_amd/synth.py`, drawn on the GPU: fp16 activations with lognormal channel scales, weights of
N(0, 0.02) rounded to nearest per output channel, the static step from a separate calibration batch.

Fields of a case: kind (which entry point), M tokens, K input channels, N output channels, h rotation block (1 = none).

  linear      pq_linear on packed nibbles, with a workspace that also holds the planes of a split product
  linear2     pq_linear2: two matrices on the same tokens (gate and up)
  linear_f6   pq_linear_f6 on weights prepacked for the 6-bit matrix instruction
  linear2_f6  pq_linear2_f6: gate and up on prepacked weights
  w4a8        pq_linear_w4a8: static 8-bit activations
  dynamic     pq_linear_dynamic: one step per token, 4 bits
  mlp_down    pq_silu_mul_rotate_quant, then pq_w4a4_gemm: the input of down_proj formed in the quantizer
"""

from __future__ import annotations

import math

import torch

import paper_2410_05265_amd.binding as pq

_CAL_TOKENS = 256


def listed():
    return [
        # one decoded token through the smallest linear of an 8B block: the call where launch and host time count most
        {"name": "decode_o", "kind": "linear", "M": 1, "K": 4096, "N": 4096, "h": 1},
        # one decoded token through gate and up of a 70B block: 235 MB of weights, the pure stream
        {"name": "decode_gate_up_70b", "kind": "linear2", "M": 1, "K": 8192, "N": 28672, "h": 1},
        # a small decode batch of an odd size (speculative or batched decoding)
        {"name": "batch_gate", "kind": "linear", "M": 13, "K": 4096, "N": 14336, "h": 1},
        # a serving batch in the middle between decode and prefill, the longest rows of the 8B block, rotated online
        {"name": "serving_down", "kind": "linear", "M": 64, "K": 14336, "N": 4096, "h": 128},
        # a larger serving batch that fills no tile evenly
        {"name": "serving_qkv", "kind": "linear", "M": 200, "K": 4096, "N": 6144, "h": 1},
        # a chunk of a chunked prefill on prepacked weights, ragged
        {"name": "chunk_o_f6", "kind": "linear_f6", "M": 333, "K": 4096, "N": 4096, "h": 1},
        # the 2048-token prefill of the paper: gate and up of an 8B block on prepacked weights
        {"name": "prefill_gate_up_f6", "kind": "linear2_f6", "M": 2048, "K": 4096, "N": 14336, "h": 1},
        # a prompt of an odd length through a 7B block's fused qkv behind the full 4096-point rotation
        {"name": "prefill_qkv_rot_f6", "kind": "linear_f6", "M": 1111, "K": 4096, "N": 12288, "h": 4096},
        # the largest single linear: down_proj of a 70B block at 2048 tokens, 128-point rotation blocks
        {"name": "prefill_down_70b_f6", "kind": "linear_f6", "M": 2048, "K": 28672, "N": 8192, "h": 128},
        # the W4A8 setting: down_proj of a 7B block for a prompt of 1500 tokens
        {"name": "w4a8_down", "kind": "w4a8", "M": 1500, "K": 11008, "N": 4096, "h": 128},
        # the per-token dynamic setting (O1): gate_proj of a 7B block behind the full rotation
        {"name": "dynamic_gate", "kind": "dynamic", "M": 777, "K": 4096, "N": 11008, "h": 4096},
        # the fused MLP tail on packed nibbles: silu(gate) * up, rotation and quantizer in one launch, then the product
        {"name": "mlp_down", "kind": "mlp_down", "M": 2048, "K": 14336, "N": 4096, "h": 128},
    ]


# token range, largest K * N, and the rotation blocks that are drawn for each kind of call
_RANGES = {
    "linear": (1, 512, 28672 * 8192, (1, 1, 128)),
    "linear2": (1, 64, 28672 * 8192, (1,)),
    "linear_f6": (128, 8192, 28672 * 8192, (1, 128, 4096)),
    "linear2_f6": (128, 4096, 14336 * 8192, (1,)),
    "w4a8": (64, 4096, 14336 * 8192, (1, 128)),
    "dynamic": (64, 4096, 14336 * 8192, (1, 4096)),
    "mlp_down": (64, 4096, 14336 * 8192, (128,)),
}


def _log_between(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    """A case of one of the listed kinds: token counts, rows and channels over their whole ranges."""
    kind = rng.choice(["linear", "linear", "linear", "linear2", "linear_f6", "linear_f6", "linear_f6", "linear2_f6",
                       "w4a8", "dynamic", "mlp_down"])
    m_lo, m_hi, kn_max, blocks = _RANGES[kind]
    h = rng.choice(blocks)
    while True:
        M = int(round(_log_between(rng, m_lo, m_hi)))
        k_step = max(h, 128)                                          # whole rotation blocks
        K = int(_log_between(rng, 2048, 28672)) // k_step * k_step
        N = int(_log_between(rng, 1024, 28672)) // 16 * 16            # any multiple of 16, not only of a tile
        outs = 2 if kind.startswith("linear2") else 1
        # no more work than the largest listed case in either unit
        if K >= k_step and K * N <= kn_max and outs * M * K * N <= 2048 * 28672 * 8192 and outs * M * N <= 2048 * 28672 * 2:
            return {"kind": kind, "M": M, "K": K, "N": N, "h": h}


# ---------------------------------------------------------------------------------------------- inputs
def _hadamard(h, dtype):
    H = torch.ones((1, 1), dtype=dtype, device="cuda")
    while H.shape[0] < h:
        H = torch.cat([torch.cat([H, H], 1), torch.cat([H, -H], 1)], 0)
    return H


def _rotate(y, h):
    """Block Hadamard rotation in y's own type (float32 for the calibration step, float64 for the exact result)."""
    if h <= 1:
        return y
    return (y.reshape(-1, h) @ _hadamard(h, y.dtype)).reshape(y.shape) / math.sqrt(h)


def _weights(gen, N, K):
    """fp16 weights of N(0, 0.02), symmetric round to nearest per output channel: packed nibbles and steps."""
    packed = torch.empty((N, K // 2), dtype=torch.uint8, device="cuda")
    steps = torch.empty((N,), dtype=torch.float32, device="cuda")
    rows = max(1, (1 << 25) // K)
    for r in range(0, N, rows):
        n = min(rows, N - r)
        w = (torch.randn((n, K), generator=gen, device="cuda") * 0.02).half().float()
        s = w.abs().amax(1) / 7.0
        q = (w / s[:, None]).round_().clamp_(-8, 7).to(torch.int8)
        packed[r:r + n] = ((q[:, 0::2] & 15) | (q[:, 1::2] << 4)).view(torch.uint8)
        steps[r:r + n] = s
    return packed, steps


def _inputs(case, seed):
    """Everything drawn from the seed: activations, static step, packed weights and their steps."""
    M, K, N, kind = case["M"], case["K"], case["N"], case["kind"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1000003 * (seed + 1))
    c = torch.exp(0.5 * torch.randn((K,), generator=gen, device="cuda"))

    def tokens(count):
        return (torch.randn((count, K), generator=gen, device="cuda") * c).half()

    d = {"x": tokens(M)}
    cal = tokens(_CAL_TOKENS).float()
    if kind == "mlp_down":
        d["up"] = tokens(M)
        cal = torch.nn.functional.silu(cal) * tokens(_CAL_TOKENS).float()
    qmax = 127.0 if kind == "w4a8" else 7.0
    d["step"] = float((_rotate(cal, case["h"]).abs().amax() / qmax).item())
    d["w"] = [_weights(gen, N, K) for _ in range(2 if kind.startswith("linear2") else 1)]
    return d


def prepare(case, seed):
    M, K, N, h, kind = case["M"], case["K"], case["N"], case["h"], case["kind"]
    d = _inputs(case, seed)
    s = {"kind": kind, "h": h, "x": d["x"], "step": d["step"], "sw": [w[1] for w in d["w"]]}
    prepacked = kind.endswith("_f6")
    s["w"] = [pq.pq_prepack_weights(w[0]) if prepacked else w[0] for w in d["w"]]
    s["out"] = [torch.empty((M, N), dtype=torch.float16, device="cuda") for _ in d["w"]]
    need = 0
    if kind in ("linear", "linear2"):
        need = pq.pq_linear_workspace_bytes_split(M, N, K)
    elif prepacked:
        need = pq.pq_linear_f6_workspace_bytes(M, K, h)
    elif kind == "w4a8":
        need = pq.pq_linear_w4a8_workspace_bytes_split(M, N, K)
    elif kind == "dynamic":
        need = pq.pq_linear_dynamic_workspace_bytes_split(M, N, K, 4)
    if need:
        s["ws"] = torch.empty((max(need, 256),), dtype=torch.uint8, device="cuda")
    if kind == "mlp_down":
        s["up"] = d["up"]
        s["codes"] = torch.empty((M, K // 2), dtype=torch.uint8, device="cuda")
    return s


def run(s):
    kind, x, w, sw, out = s["kind"], s["x"], s["w"], s["sw"], s["out"]
    if kind == "linear":
        return pq.pq_linear(x, w[0], sw[0], s["step"], s["h"], out=out[0], workspace=s["ws"])[0]
    if kind == "linear2":
        return pq.pq_linear2(x, w[0], sw[0], w[1], sw[1], s["step"], s["h"], out_a=out[0], out_b=out[1],
                             workspace=s["ws"])[:2]
    if kind == "linear_f6":
        return pq.pq_linear_f6(x, w[0], sw[0], s["step"], s["h"], out=out[0], workspace=s["ws"])[0]
    if kind == "linear2_f6":
        return pq.pq_linear2_f6(x, w[0], sw[0], w[1], sw[1], s["step"], s["h"], out_a=out[0], out_b=out[1],
                                workspace=s["ws"])[:2]
    if kind == "w4a8":
        return pq.pq_linear_w4a8(x, w[0], sw[0], s["step"], s["h"], out=out[0], workspace=s["ws"])[0]
    if kind == "dynamic":
        return pq.pq_linear_dynamic(x, w[0], sw[0], s["h"], 1.0, 4, out=out[0], workspace=s["ws"])[0]
    codes = pq.pq_silu_mul_rotate_quant(x, s["up"], s["h"], s["step"], out=s["codes"])
    return codes, pq.pq_w4a4_gemm(codes, w[0], sw[0], s["step"], out=out[0])[0]


# ---------------------------------------------------------------------------------------- what is needed
def work(case):
    M, K, N, kind = case["M"], case["K"], case["N"], case["kind"]
    mats = 2 if kind.startswith("linear2") else 1
    per_weight = 0.75 if kind.endswith("_f6") else 0.5          # bytes of a weight in the form the call takes
    nbytes = 2.0 * M * K + mats * (per_weight * N * K + 4.0 * N + 2.0 * M * N)
    if kind == "mlp_down":
        nbytes += 2.0 * M * K + M * K / 2                       # the second producer input, and the codes it returns
    return {"bytes": nbytes, "flops": 2.0 * mats * M * N * K}


def tolerance(case):
    """fp16 outputs of exact integer sums.  Without rotation another implementation differs by the last bit of an
    fp16 result at most (2-norm error of one fp16 rounding: 2e-4).  With rotation (or a dynamic step, or silu) the
    fp32 sums of another order move some codes across a rounding tie: each moves its token's outputs by one step
    of the activation times a weight code, about 8 / (1.7 * 2.5 sqrt(K)) of their rms at most."""
    if case["h"] <= 1 and case["kind"] not in ("dynamic", "mlp_down"):
        return {"rel": 1e-3, "max": 4e-3}
    # (a code flips where |y / s - (k + 1/2)| is below the fp32 error of y: a share of about 1e-6 of them.  Measured
    # against 64 bits: 4e-4 behind a rotation, 7e-4 behind silu, whose exponential is the hardware's)
    return {"rel": 3e-3 if case["kind"] == "mlp_down" else 2e-3, "max": 0.15, "differ": 2e-5}


# -------------------------------------------------------------------------------------- the 64-bit result
def _unpack(packed):
    lo = (packed << 4).view(torch.int8) >> 4
    hi = packed.view(torch.int8) >> 4
    return torch.stack([lo, hi], -1).reshape(packed.shape[0], -1)


def exact(case, seed):
    kind, h = case["kind"], case["h"]
    d = _inputs(case, seed)
    y = d["x"].double()
    if kind == "mlp_down":
        y = y / (1.0 + torch.exp(-y)) * d["up"].double()
    y = _rotate(y, h)
    if kind == "dynamic":
        step = (y.abs().amax(1, keepdim=True) / 7.0).float().double()
        step = torch.where(step > 0, step, torch.ones_like(step))
    else:
        step = float(torch.tensor(d["step"], dtype=torch.float32).double())
    lo, hi = (-128, 127) if kind == "w4a8" else (-8, 7)
    q = (y / step).round_().clamp_(lo, hi)
    outs = []
    for packed, sw in d["w"]:
        out = torch.empty((case["M"], case["N"]), dtype=torch.float64, device="cuda")
        for r in range(0, case["N"], 4096):
            out[:, r:r + 4096] = q @ _unpack(packed[r:r + 4096]).double().t().contiguous()
        outs.append(out * step * sw.double())
    if kind == "mlp_down":
        c = q.to(torch.int8)
        return ((c[:, 0::2] & 15) | (c[:, 1::2] << 4)).view(torch.uint8), outs[0]
    return tuple(outs) if kind.startswith("linear2") else outs[0]
