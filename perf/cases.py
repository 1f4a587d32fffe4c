"""What a program that uses this library has it do, as cases to be timed: C = A B + C through the
Python binding of the C ABI, over the library's whole range -- the smallest calls (one 256 x 256
result), ordinary squares and transformer shapes, the largest square of the sweep, ragged and odd
sizes, few rows against a large matrix -- in the modes it has: f32 C, f16 C, f16 C with lent
scratch memory, and each of the first two with the fused bias and ReLU.

Operands are drawn on the GPU from the distributions of `paper_2108_13191_amd.workloads`.
"""
import math

import torch

from paper_2108_13191_amd import binding

# mode: "f32" / "f16": gemm_f16_f32acc / gemm_f16_f16acc; "f16ws": gemm_f16_f16acc_workspace.
# fused: bias and ReLU through the _bias_act entry point of the mode.  dist: distribution of A, B.
# c: that of the old C.  pad: elements between the rows' ends and the pitches of A, B and C.


def _case(name, M, N, K, mode, dist, c="zeros", fused=False, pad=0):
    d = {"M": M, "N": N, "K": K, "mode": mode, "dist": dist, "c": c, "fused": fused, "pad": pad}
    return dict(d, name=name) if name else d


def listed():
    return [
        # the smallest named problem: launch and latency
        _case("sq256_f32", 256, 256, 256, "f32", "uniform"),
        # small squares: fewer results than fill the chip with large tiles; f16 C with an old value
        _case("sq1024_f16", 1024, 1024, 1024, "f16", "normal_rsqrtk", c="uniform"),
        _case("sq2048_f32", 2048, 2048, 2048, "f32", "uniform"),
        # the headline square, and the largest one of the sweep in the half-precision mode
        _case("sq8192_f32", 8192, 8192, 8192, "f32", "normal_rsqrtk"),
        _case("sq16384_f16", 16384, 16384, 16384, "f16", "normal_rsqrtk"),
        # transformer layers over 16384 tokens: FFN up with its bias and ReLU in f16, FFN down, QKV
        _case("ffn_up_bias_relu_f16", 16384, 3072, 768, "f16", "normal_0p02", fused=True),
        _case("ffn_down_f32", 16384, 768, 3072, "f32", "normal_0p02"),
        _case("qkv_f32", 16384, 2304, 768, "f32", "normal_0p02"),
        # no multiple of any tile, still aligned
        _case("ragged4000_f32", 4000, 4000, 4000, "f32", "normal_0p02"),
        # no alignment at all: odd sizes and odd pitches
        _case("odd2001_f32", 2001, 1999, 2003, "f32", "normal_0p02", c="uniform"),
        # decoding: a few rows against a large weight matrix; a small batch with scratch memory lent
        _case("skinny16_f16", 16, 8192, 8192, "f16", "normal_0p02"),
        _case("skinny256_f16ws", 256, 4096, 16384, "f16ws", "normal_0p02"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: general sizes from 64 to 16384 (aligned or odd), transformer-like shapes of
    many rows, or skinny problems of 1 to 256 rows (or columns); any mode that fits."""
    while True:
        kind = rng.choice(["general", "general", "rows", "skinny"])
        odd = rng.random() < 0.35
        if kind == "general":
            M, N, K = (_log(rng, 64, 16384) for _ in range(3))
        elif kind == "rows":
            M, N, K = _log(rng, 2048, 16384), _log(rng, 512, 8192), _log(rng, 256, 4096)
        else:
            M, N, K = _log(rng, 1, 256), _log(rng, 1024, 16384), _log(rng, 1024, 16384)
            if rng.random() < 0.25:
                M, N = N, max(8, M)
        if odd:
            pad = rng.choice([0, 0, 1, 3])
        else:
            N, K = max(8, N // 8 * 8), max(8, K // 8 * 8)
            pad = rng.choice([0, 0, 0, 8, 64])
        mode = rng.choice(["f32", "f32", "f16", "f16ws"] if kind == "skinny" else ["f32", "f16"])
        fused = mode != "f16ws" and rng.random() < 0.25
        dist = rng.choice(["normal_rsqrtk", "normal_0p02"])
        # no drawn case costs more than the largest listed one (without alignment a product costs more)
        if M * N * K <= (4096 ** 3 if odd else 16384 ** 3):
            return _case(None, M, N, K, mode, dist, rng.choice(["zeros", "uniform"]), fused, pad)


def _matrix(rows, cols, ld, dist, dtype, K, gen):
    m = torch.empty((rows, ld), dtype=dtype, device="cuda")[:, :cols]
    if dist == "zeros":
        return m.zero_()
    x = torch.empty((rows, cols), dtype=torch.float32, device="cuda")
    if dist == "uniform":
        x.uniform_(-1.0, 1.0, generator=gen)
    else:
        x.normal_(0.0, 0.02 if dist == "normal_0p02" else K ** -0.5, generator=gen)
    return m.copy_(x)


def prepare(case, seed):
    M, N, K, pad = case["M"], case["N"], case["K"], case["pad"]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    c_type = torch.float32 if case["mode"] == "f32" else torch.float16
    s = {
        "size": (M, N, K), "mode": case["mode"], "fused": case["fused"],
        "A": _matrix(M, K, K + pad, case["dist"], torch.float16, K, gen), "lda": K + pad,
        "B": _matrix(K, N, N + pad, case["dist"], torch.float16, K, gen), "ldb": N + pad,
        "C": _matrix(M, N, N + pad, case["c"], c_type, K, gen), "ldc": N + pad,
        "stream": torch.cuda.current_stream().cuda_stream,
    }
    if case["fused"]:
        s["bias"] = _matrix(1, N, N, "normal_0p02", c_type, K, gen)
    if case["mode"] == "f16ws":
        need = binding.gemm_f16_f16acc_workspace_bytes(M, N, K)
        s["workspace"] = torch.empty(max(need, 16), dtype=torch.uint8, device="cuda")
        s["workspace_bytes"] = need
    return s


def run(s):
    M, N, K = s["size"]
    operands = (M, N, K, s["A"], s["lda"], s["B"], s["ldb"], s["C"], s["ldc"])
    if s["fused"]:
        f = binding.gemm_f16_f32acc_bias_act if s["mode"] == "f32" else binding.gemm_f16_f16acc_bias_act
        rc = f(*operands, s["bias"], binding.ACT_RELU, s["stream"])
    elif s["mode"] == "f16ws":
        rc = binding.gemm_f16_f16acc_workspace(*operands, s["workspace"], s["workspace_bytes"], s["stream"])
    else:
        f = binding.gemm_f16_f32acc if s["mode"] == "f32" else binding.gemm_f16_f16acc
        rc = f(*operands, s["stream"])
    binding.check(rc)
    return s["C"]


def work(case):
    M, N, K = case["M"], case["N"], case["K"]
    c_size = 4 if case["mode"] == "f32" else 2
    return {"bytes": 2 * (M * K + K * N) + 2 * M * N * c_size + (N * c_size if case["fused"] else 0), "flops": 2 * M * N * K}


def tolerance(case):
    """Largest relative error between two correct implementations, from comparing the results with
    ones formed in 64 bits (two passes, the second on the first's C), times about four: f32 sums
    of any order (seen: 6e-7 and 4.5e-6, at K = 8192); in f16 mode one rounding to 11 bits per
    pass (seen: 2.1e-4 and 4.9e-4)."""
    if case["mode"] == "f32":
        return {"rel": 2.5e-6, "max": 2e-5}
    return {"rel": 8e-4, "max": 2e-3}
