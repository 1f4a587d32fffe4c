"""The 128 x 128 kernel whose two groups of wavefronts take the k steps in turn: its loops left at every exit (0 to 13 whole
k steps, with and without a k tail), edge tiles beside whole ones, both types of C, a pitch of C that is not N; integers
bit for bit against the oracle, NaN around A and B; and problems that automatic selection gives it, alone and as the second of two launches."""
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
NAME = "pp128x128x64_w2x2_k2"


@pytest.fixture(autouse=True)
def _unforce():
    yield
    binding.force_config(-1)


@pytest.mark.parametrize("tail", [0, 8, 40])
def test_every_exit_of_the_k_loop(oracle_mod, tail):
    binding.force_config(config_id(NAME))
    for steps in range(0, 14):
        K = 64 * steps + tail
        if K == 0:
            continue
        M, N = ((128, 128), (129, 264), (300, 136))[steps % 3]
        mode = ("f32", "f16")[(steps + tail // 8) % 2]
        A, B, _ = wl.make_inputs(M, N, K, "int2", "zeros", seed=10400 + K)
        C0 = np.random.default_rng(K).integers(-4, 5, size=(M, N)).astype(CDT[mode])
        got = run_gemm(A, B, C0, mode, lda=K + 8 * (steps % 2), ldb=N + 16, ldc=N + 5, offs=(0, 0, 1))
        Cref, _ = oracle_mod.gemm_f16(A, B, C0)
        want = oracle_mod.round_to_f32(Cref) if mode == "f32" else Cref.astype(np.float16)
        assert np.array_equal(got, want), (M, N, K, mode)


@pytest.mark.parametrize("tail", [0, 40])
def test_loops_that_request_c_among_their_copies(oracle_mod, tail):
    """14 to 21 whole k steps: the main loop runs, for both groups from 15 on, and either group leaves it at either parity."""
    binding.force_config(config_id(NAME))
    for steps in range(14, 22):
        K = 64 * steps + tail
        M, N = ((256, 128), (130, 272), (300, 136))[steps % 3]
        mode = ("f32", "f16")[steps // 2 % 2]
        A, B, _ = wl.make_inputs(M, N, K, "int2", "zeros", seed=10450 + K)
        C0 = np.random.default_rng(K).integers(-4, 5, size=(M, N)).astype(CDT[mode])
        got = run_gemm(A, B, C0, mode, ldc=N + 3, offs=(0, 0, 1))
        Cref, _ = oracle_mod.gemm_f16(A, B, C0)
        want = oracle_mod.round_to_f32(Cref) if mode == "f32" else Cref.astype(np.float16)
        assert np.array_equal(got, want), (M, N, K, mode)


def test_selected(oracle_mod):
    M, N, K = 2048, 1920, 2048
    assert binding.query_config(0, M, N, K, 16, K, 16, N, 16, N)["name"] == NAME
    assert binding.query_config(0, M, N, K, 16, K + 8, 16, N, 16, N)["name"] != NAME           # rows that begin within a line
    A, B, C0 = wl.make_inputs(M, N, K, "normal_0p02", "uniform", seed=10500)
    got = run_gemm(A, B, C0, "f32")
    rows = np.array([0, 1, 127, 128, 1000, 2047])
    Cref, S = oracle_mod.gemm_f16(A, B, C0, rows=rows)
    assert_close(got[rows], Cref, S, C0[rows], "f32", what=NAME)


def test_selected_for_left_over_rows(oracle_mod):
    """f16 mode: the rows behind a first launch of 256 x 256 tiles, edge tiles among them, and the rows next to them; integers, bit for bit."""
    M, N, K = 2501, 7360, 832
    q = binding.query_config(1, M, N, K, 16, K, 16, N, 16, N)
    assert q["split_rows"] == 2048 and binding.describe_config(q["id2"])["name"] == NAME
    A, B, C0 = wl.make_inputs(M, N, K, "int1", "zeros", seed=10600, c_dtype=np.float16)
    C0[:] = (np.arange(M)[:, None] + np.arange(N)[None, :]) % 5 - 2
    got = run_gemm(A, B, C0, "f16")
    rows = np.array([0, 2046, 2047, 2048, 2049, 2111, 2112, 2175, 2176, 2431, 2432, 2499, 2500])
    Cref, _ = oracle_mod.gemm_f16(A, B, C0, rows=rows)
    assert np.array_equal(got[rows], Cref.astype(np.float16))
