"""Operands of any alignment: the 128 x 128 kernel in both its forms (one and two k groups), forced -- edges
of its tiles and of its 8-element chunks (a chunk past the end of a row is loaded as the row's
last 8 elements and what is there twice is zeroed), every remainder of its k steps, both types of C, the
fused epilogue, infinities in the tail -- and what automatic selection runs on such problems, the small
tiles among it.  Integers bit for bit against the oracle (every partial sum is exact); NaN around A
and B would show any read outside them."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from gpu_util import DevMat, assert_close, config_id, run_gemm
from paper_2108_13191_amd import binding
from paper_2108_13191_amd import workloads as wl

pytestmark = pytest.mark.gpu
CDT = {"f32": np.float32, "f16": np.float16}
FORMS = ["generic128x128x64", "generic128x128x64_k2"]


@pytest.fixture(autouse=True)
def _unforce():
    yield
    binding.force_config(-1)


def _force(name, M, N, K):
    binding.force_config(config_id(name))
    assert binding.query_config(False, M, N, K, 2, K, 2, N, 4, N)["name"] == name


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


@pytest.mark.parametrize("name", FORMS)
def test_forced_tile_and_chunk_edges(oracle_mod, name):
    _force(name, 127, 17, 9)
    for i, N in enumerate((8, 9, 15, 17, 121, 127, 128, 129, 136, 255, 263)):
        for j, M in enumerate((1, 127, 129)):
            for odd in (0, 1):
                _ints(oracle_mod, M, N, (8, 9, 65, 200)[(i + j) % 4], ("f32", "f16")[(i + j + odd) % 2], seed=9500 + 10 * i + j, offs=(odd, 1, odd), pads=(1, odd, 3))


@pytest.mark.parametrize("name", FORMS)
def test_forced_every_remainder_of_the_k_steps(oracle_mod, name):
    _force(name, 130, 141, 65)
    for steps in range(0, 11):
        for tail in (0, 1, 8, 39, 63):
            K = 64 * steps + tail
            if K >= 8:
                _ints(oracle_mod, 130, 141, K, ("f32", "f16")[(steps + tail) % 2], seed=9600 + K, pads=(tail % 2, 3, 1))


@pytest.mark.parametrize("mode", ["f32", "f16"])
@pytest.mark.parametrize("name", FORMS)
def test_forced_random_data_fused_epilogue_and_infinities(oracle_mod, name, mode):
    M, N, K = 200, 203, 333
    _force(name, M, N, K)
    A, B, C0 = wl.make_inputs(M, N, K, "uniform", "uniform", seed=9700, c_dtype=CDT[mode])
    got = run_gemm(A, B, C0, mode, lda=K + 1, offs=(1, 0, 0))
    Cref, S = oracle_mod.gemm_f16(A, B, C0)
    assert_close(got, Cref, S, C0, mode, what=name)
    # bias and ReLU, integers
    Ai, Bi, _ = wl.make_inputs(M, N, K, "int2", "zeros", seed=9701)
    Ci = np.random.default_rng(2).integers(-4, 5, size=(M, N)).astype(CDT[mode])
    bias = (np.arange(N) % 13 - 6).astype(CDT[mode])
    dA, dB, dC, db = DevMat(Ai, K + 1, 1, nan_canary=True), DevMat(Bi, N + 2, 1, nan_canary=True), DevMat(Ci, N + 1, 1), torch.from_numpy(bias).cuda()
    f = binding.gemm_f16_f32acc_bias_act if mode == "f32" else binding.gemm_f16_f16acc_bias_act
    binding.check(f(M, N, K, dA.ptr, dA.ld, dB.ptr, dB.ld, dC.ptr, dC.ld, db, binding.ACT_RELU, torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    Cref, _ = oracle_mod.gemm_f16(Ai, Bi, Ci)
    assert np.array_equal(dC.fetch(), np.maximum(Cref + bias[None, :], 0).astype(CDT[mode]))
    # infinities and zeros among the last 8 k
    A[3, K - 2] = np.inf
    B[K - 5, 7] = -np.inf
    B[K - 2, 100] = 0.0                                   # inf * 0 = NaN at (3, 100)
    C0[5, 5] = np.nan
    with np.errstate(invalid="ignore", over="ignore"):
        got = run_gemm(A, B, C0, mode).astype(np.float64)
        Cref, _ = oracle_mod.gemm_f16(A, B, C0)
    for pick in (np.isnan, np.isposinf, np.isneginf):
        assert np.array_equal(pick(got), pick(Cref))
    assert np.isnan(got[3, 100]) and np.isnan(got[5, 5])


@pytest.mark.parametrize("name", FORMS + ["ks16x32x64_k8", "ks64x64x64_k8"])
def test_largest_pitch_and_offsets_beyond_4_gb(oracle_mod, name):
    """A pitch of 2^22 elements, the largest that these kernels take: A, B and C each span more than 4 GB, and
    byte offsets within a tile reach 2^30."""
    ld, M, N, K = 1 << 22, 521, 25, 523
    A, B, _ = wl.make_inputs(M, N, K, "int2", "zeros", seed=9800)
    C0 = np.random.default_rng(4).integers(-4, 5, size=(M, N)).astype(np.float32)
    binding.force_config(config_id(name))
    assert binding.query_config(False, M, N, K, 2, ld, 2, ld, 4, ld)["name"] in (name, "generic_" + name)

    def put(x, dtype):
        t = torch.empty((x.shape[0] - 1) * ld + x.shape[1], dtype=dtype, device="cuda")      # exactly the matrix
        v = torch.as_strided(t, x.shape, (ld, 1))
        v.copy_(torch.from_numpy(x))
        return t, v
    (a, _), (b, _), (c, cv) = put(A, torch.float16), put(B, torch.float16), put(C0, torch.float32)
    binding.check(binding.gemm_f16_f32acc(M, N, K, a, ld, b, ld, c, ld, torch.cuda.current_stream().cuda_stream))
    got = cv.contiguous().cpu().numpy()
    Cref, _ = oracle_mod.gemm_f16(A, B, C0)
    assert np.array_equal(got, oracle_mod.round_to_f32(Cref))


def test_what_runs():
    q = binding.query_config(False, 500, 501, 503, 2, 503, 2, 501, 4, 501)
    assert q["id"] == 0 and q["name"] == "generic_ks32x32x64_k8"
    assert binding.query_config(False, 2001, 1999, 2003, 2, 2003, 2, 1999, 4, 1999)["name"] == "generic128x128x64_k2"
    assert binding.query_config(False, 2177, 2049, 391, 2, 391, 2, 2049, 4, 2049)["name"] == "generic128x128x64"
    for M, N, K in ((500, 7, 503), (500, 501, 7)):        # no chunk of 8 elements: element by element
        assert binding.query_config(False, M, N, K, 2, K, 2, N, 4, N)["block_m"] == 64
