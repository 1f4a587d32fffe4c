"""The tiled kernel for operands of any alignment: edges of its tiles and of its 8-element chunks
(a chunk past the end of a row is loaded as the row's last 8 elements and what is there twice is
zeroed), every remainder of its k steps, one and two k groups.  Integers bit for bit against the
oracle (every partial sum is exact); NaN around A and B would show any read outside them."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from gpu_util import assert_close, run_gemm
from paper_2108_13191_amd import binding
from paper_2108_13191_amd import workloads as wl

pytestmark = pytest.mark.gpu
CDT = {"f32": np.float32, "f16": np.float16}


def _ints(oracle_mod, M, N, K, mode, seed, offs=(1, 1, 1), pads=(1, 3, 1)):
    A, B, _ = wl.make_inputs(M, N, K, "int2", "zeros", seed=seed)
    C0 = np.random.default_rng(seed).integers(-4, 5, size=(M, N)).astype(CDT[mode])
    got = run_gemm(A, B, C0, mode, lda=K + pads[0], ldb=N + pads[1], ldc=N + pads[2], offs=offs)
    Cref, _ = oracle_mod.gemm_f16(A, B, C0)
    want = oracle_mod.round_to_f32(Cref) if mode == "f32" else Cref.astype(np.float16)
    assert np.array_equal(got, want), (M, N, K, mode)


@pytest.mark.parametrize("mode", ["f32", "f16"])
def test_tile_and_chunk_edges(oracle_mod, mode):
    for i, N in enumerate((8, 9, 15, 17, 121, 127, 128, 129, 136, 255, 263)):
        for M in (1, 127, 129):
            K = (8, 9, 65)[(i + M) % 3]
            _ints(oracle_mod, M, N, K, mode, seed=9000 + 10 * i + M % 7)


def test_every_remainder_of_the_k_steps(oracle_mod):
    for K in list(range(8, 24)) + [63, 64, 65, 71, 72, 73, 127, 128, 129, 191, 193, 255, 257, 319, 321, 385, 447, 513]:
        _ints(oracle_mod, 130, 141, K, ("f32", "f16")[K % 2], seed=9200 + K)


@pytest.mark.parametrize("K", [9, 70, 129, 200, 263, 391])
def test_more_tiles_than_compute_units(oracle_mod, K):
    # 17 x 17 tiles of 128 x 128: one k group per tile
    _ints(oracle_mod, 2177, 2049, K, "f32", seed=9300 + K, pads=(0, 0, 0), offs=(0, 0, 0))


@pytest.mark.parametrize("mode", ["f32", "f16"])
def test_random_data_and_infinities_in_the_tail(oracle_mod, mode):
    M, N, K = 200, 203, 333
    A, B, C0 = wl.make_inputs(M, N, K, "uniform", "uniform", seed=9400, c_dtype=CDT[mode])
    got = run_gemm(A, B, C0, mode, lda=K + 1, offs=(1, 0, 0))
    Cref, S = oracle_mod.gemm_f16(A, B, C0)
    assert_close(got, Cref, S, C0, mode, what="unaligned")
    # an infinity in the last 8 elements of a row of A / k rows of B meets zeros only where the data has them
    A[3, K - 2] = np.inf
    B[K - 5, 7] = -np.inf
    B[K - 2, 100] = 0.0                                   # inf * 0 = NaN at (3, 100)
    with np.errstate(invalid="ignore", over="ignore"):
        got = run_gemm(A, B, C0, mode).astype(np.float64)
        Cref, S = oracle_mod.gemm_f16(A, B, C0)
    for pick in (np.isnan, np.isposinf, np.isneginf):
        assert np.array_equal(pick(got), pick(Cref))
    assert np.isnan(got[3, 100]) and np.isinf(got[:, 7]).sum() == M - np.isnan(got[:, 7]).sum()


def test_what_runs():
    q = binding.query_config(False, 500, 501, 503, 2, 503, 2, 501, 4, 501)
    assert q["id"] == 0 and q["name"].startswith("generic") and (q["block_m"], q["block_n"]) != (64, 64)
    for M, N, K in ((500, 7, 503), (500, 501, 7)):        # no chunk of 8 elements: element by element
        assert binding.query_config(False, M, N, K, 2, K, 2, N, 4, N)["block_m"] == 64
