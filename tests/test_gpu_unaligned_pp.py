"""The 256 x 256 and 128 x 256 tiles for operands of any alignment, forced: edges of their tiles and of their
8-element chunks, every exit of the k loop with and without a tail, both types of C, the fused epilogue, infinities in
the tail, the largest pitch; and what automatic selection gives them.  Integers bit for bit against the oracle (every
partial sum is exact); NaN around A and B would show any read outside them."""
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
FORMS = ["generic256x256x64", "generic128x256x64"]


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


@pytest.mark.parametrize("name", FORMS)
def test_tile_and_chunk_edges(oracle_mod, name):
    _force(name, 127, 17, 9)
    for i, N in enumerate((8, 9, 15, 17, 249, 255, 256, 257, 264, 519)):
        for j, M in enumerate((1, 127, 129, 257)):
            odd = (i + j) % 2
            _ints(oracle_mod, M, N, (8, 9, 65, 200)[(i + 2 * j) % 4], ("f32", "f16")[(i // 2 + j) % 2], seed=9900 + 10 * i + j, offs=(odd, 1, odd), pads=(1, odd, 3))


@pytest.mark.parametrize("name", FORMS)
def test_every_exit_of_the_k_loop(oracle_mod, name):
    _force(name, 130, 141, 65)
    for steps in range(0, 7):
        for tail in (0, 1, 8, 39, 63):
            K = 64 * steps + tail
            if K >= 8:
                _ints(oracle_mod, 270, 300, K, ("f32", "f16")[(steps + tail) % 2], seed=10000 + K, pads=(tail % 2, 3, 1))


@pytest.mark.parametrize("mode", ["f32", "f16"])
@pytest.mark.parametrize("name", FORMS)
def test_random_data_fused_epilogue_and_infinities(oracle_mod, name, mode):
    M, N, K = 300, 403, 333
    _force(name, M, N, K)
    A, B, C0 = wl.make_inputs(M, N, K, "uniform", "uniform", seed=10100, c_dtype=CDT[mode])
    got = run_gemm(A, B, C0, mode, lda=K + 1, offs=(1, 0, 0))
    Cref, S = oracle_mod.gemm_f16(A, B, C0)
    assert_close(got, Cref, S, C0, mode, what=name)
    # bias and ReLU, integers
    Ai, Bi, _ = wl.make_inputs(M, N, K, "int2", "zeros", seed=10101)
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


@pytest.mark.parametrize("name", FORMS)
def test_largest_pitch(oracle_mod, name):
    """A pitch of 2^22 elements: A, B and C each span more than 4 GB, and byte offsets within a tile of A reach 2^31."""
    ld, M, N, K = 1 << 22, 521, 25, 523
    A, B, _ = wl.make_inputs(M, N, K, "int2", "zeros", seed=10200)
    C0 = np.random.default_rng(4).integers(-4, 5, size=(M, N)).astype(np.float32)
    _force(name, M, N, K)

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


@pytest.mark.parametrize("M,N,K,name", [(4001, 3999, 4003, FORMS[0]), (2001, 3999, 1003, FORMS[1]), (3067, 5721, 447, "generic128x128x64")])
def test_selected_on_sampled_rows(oracle_mod, M, N, K, name):
    q = binding.query_config(False, M, N, K, 2, K, 2, N, 4, N)
    assert (q["id"], q["name"]) == (0, name)
    A, B, C0 = wl.make_inputs(M, N, K, "normal_0p02", "uniform", seed=10300)
    got = run_gemm(A, B, C0, "f32")
    rows = np.array([0, 1, 127, 128, M // 2, M - 2, M - 1])
    Cref, S = oracle_mod.gemm_f16(A, B, C0, rows=rows)
    assert_close(got[rows], Cref, S, C0[rows], "f32", what=name)
