"""The small-tile kernels whose wavefronts take the k steps in turn: edges of their tiles and of their
8-element chunks, every remainder of the k steps over the wavefronts' turns, operands of any
alignment.  Integers bit for bit against the oracle (every partial sum is exact); NaN around A and B
would show any read outside them."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from gpu_util import assert_close, config_id, run_gemm
from paper_2108_13191_amd import binding
from paper_2108_13191_amd import workloads as wl

pytestmark = pytest.mark.gpu
CDT = {"f32": np.float32, "f16": np.float16}
NAMES = ["ks16x32x64_k8", "ks32x32x64_k8", "ks16x64x64_k8", "ks32x64x64_k8", "ks64x64x64_k8"]


@pytest.fixture(autouse=True)
def _unforce():
    yield
    binding.force_config(-1)


def _ints(oracle_mod, M, N, K, mode, seed, offs=(0, 0, 0), pads=(0, 0, 0), what=""):
    A, B, _ = wl.make_inputs(M, N, K, "int2", "zeros", seed=seed)
    C0 = np.random.default_rng(seed).integers(-4, 5, size=(M, N)).astype(CDT[mode])
    got = run_gemm(A, B, C0, mode, lda=K + pads[0], ldb=N + pads[1], ldc=N + pads[2], offs=offs)
    Cref, _ = oracle_mod.gemm_f16(A, B, C0)
    want = oracle_mod.round_to_f32(Cref) if mode == "f32" else Cref.astype(np.float16)
    assert np.array_equal(got, want), (what, M, N, K, mode)


@pytest.mark.parametrize("name", NAMES)
def test_tile_and_chunk_edges(oracle_mod, name):
    binding.force_config(config_id(name))
    for i, (M, N) in enumerate([(1, 8), (15, 31), (16, 32), (17, 33), (31, 63), (33, 65), (64, 64), (65, 71), (130, 9), (48, 136)]):
        for odd in (0, 1):
            _ints(oracle_mod, M, N, (8, 9, 72, 200)[i % 4], ("f32", "f16")[(i + odd) % 2], 9500 + i, offs=(odd, odd, odd), pads=(odd, 3 * odd, 5), what=name)


@pytest.mark.parametrize("name", NAMES)
def test_every_remainder_of_the_k_steps(oracle_mod, name):
    """1 to 34 k steps over eight wavefronts (one to five turns each), whole and with tails."""
    binding.force_config(config_id(name))
    for steps in range(0, 34):
        K = 64 * steps + (0 if steps % 3 == 1 else 8 + 5 * (steps % 11))
        _ints(oracle_mod, 40, 72, K, ("f32", "f16")[steps % 2], 9600 + steps, what=name)


@pytest.mark.parametrize("mode", ["f32", "f16"])
def test_selected_for_small_results_and_right_there(oracle_mod, mode):
    """Under automatic selection, aligned and odd; random data, NaN and infinities."""
    for (M, N, K) in [(256, 256, 256), (1024, 1024, 512), (100, 3000, 704), (3, 1160, 1688), (201, 203, 1333), (1, 2049, 2047)]:
        q = binding.query_config(mode == "f16", M, N, K, 16, K, 16, N, 16, N)
        assert "ks" in q["name"] and q["grid"] >= 1, q
        A, B, C0 = wl.make_inputs(M, N, K, "uniform", "uniform", seed=K, c_dtype=CDT[mode])
        got = run_gemm(A, B, C0, mode)
        Cref, S = oracle_mod.gemm_f16(A, B, C0)
        assert_close(got, Cref, S, C0, mode, what=f"small tiles {(M, N, K)} {mode}")
    M, N, K = 40, 75, 333
    A, B, C0 = wl.make_inputs(M, N, K, "uniform", "uniform", seed=11, c_dtype=CDT[mode])
    A[3, K - 2] = np.inf
    B[K - 5, 7] = -np.inf
    B[K - 2, 60] = 0.0                                    # inf * 0 = NaN at (3, 60)
    C0[5, 5] = np.nan
    with np.errstate(invalid="ignore", over="ignore"):
        got = run_gemm(A, B, C0, mode).astype(np.float64)
        Cref, _ = oracle_mod.gemm_f16(A, B, C0)
    for pick in (np.isnan, np.isposinf, np.isneginf):
        assert np.array_equal(pick(got), pick(Cref))


def test_fused_epilogue_at_odd_sizes(oracle_mod):
    M, N, K = 50, 77, 190
    A, B, _ = wl.make_inputs(M, N, K, "int2", "zeros", seed=12)
    for mode in ("f32", "f16"):
        C0 = np.random.default_rng(1).integers(-4, 5, size=(M, N)).astype(CDT[mode])
        bias = (np.arange(N) % 13 - 6).astype(CDT[mode])
        dA, dB, dC, db = (torch.from_numpy(x).cuda() for x in (A, B, C0, bias))
        f = binding.gemm_f16_f32acc_bias_act if mode == "f32" else binding.gemm_f16_f16acc_bias_act
        binding.check(f(M, N, K, dA, K, dB, N, dC, N, db, binding.ACT_RELU, torch.cuda.current_stream().cuda_stream))
        torch.cuda.synchronize()
        Cref, _ = oracle_mod.gemm_f16(A, B, C0)
        assert np.array_equal(dC.cpu().numpy(), np.maximum(Cref + bias[None, :], 0).astype(CDT[mode]))
