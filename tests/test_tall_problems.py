"""Many rows and few columns, or few rows, long k loops: the small tiles on as many workgroups as there are tiles (no split k
loop in the f32 mode, no limit by the count of 64 x 64 tiles in the f16 mode), where the estimates say so."""
import numpy as np
import pytest

from paper_2108_13191_amd import binding
from paper_2108_13191_amd import workloads as wl

SHAPES = [(2541, 8, 2280), (598, 72, 2312), (1753, 8, 9784), (3306, 184, 2096), (5000, 32, 2048)]
# up to 32 columns on the small tiles, one round of 32 x 32 or a second one well filled
NARROW = [(1257, 16, 5544), (479, 8, 7872), (129, 32, 8704), (8192, 24, 2048), (12000, 16, 2176)]
FEW = [(1, 3192, 2208), (10, 1072, 5672), (89, 96, 11496), (160, 760, 3496)]
WIDE = [(127, 1120, 2384), (16, 2048, 2048)]


def _name(f16, M, N, K):
    return binding.query_config(f16, M, N, K, 16, K, 16, N, 16, N)["name"]


def test_what_runs():
    for f16, shapes in ((0, [SHAPES[0], SHAPES[1], SHAPES[4]]), (1, [SHAPES[0], SHAPES[1], SHAPES[2], SHAPES[4]])):
        for M, N, K in shapes:
            q = binding.query_config(f16, M, N, K, 16, K, 16, N, 16, N)
            assert q["name"].startswith("ks") and q["grid"] > ((M + 63) // 64) * ((N + 63) // 64), (f16, M, N, K, q)
    assert _name(0, 3306, 184, 2096).startswith("ks") and _name(0, 184, 1120, 2384).startswith("ks")
    # few rows, or one tile either way, in the f16 mode; the f32 mode where B is not latency-bound
    for M, N, K in FEW:
        q = binding.query_config(1, M, N, K, 16, K, 16, N, 16, N)
        assert q["name"].startswith("ks") and q["grid"] > ((M + 63) // 64) * ((N + 63) // 64), (M, N, K, q)
    assert _name(0, 1, 3192, 2208).startswith("ks") and _name(0, 14, 1640, 4976) == "w4a_128x128x64"


def test_narrow_problems():
    """f32 mode, up to 32 columns: small tiles up to K = 8704; cut along k beyond, with 40 columns
    (by the estimates) and where a second round of the small tiles would be nearly empty."""
    for M, N, K in NARROW:
        assert _name(0, M, N, K).startswith("ks"), (M, N, K)
    for M, N, K in [(334, 24, 15880), (129, 32, 8712), (9421, 16, 8512), (512, 40, 8192), (8200, 16, 8192)]:
        assert _name(0, M, N, K) == "w4a_128x128x64", (M, N, K)


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", SHAPES + FEW + WIDE + NARROW)
def test_results(oracle_mod, M, N, K):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from gpu_util import assert_close, run_gemm
    for mode, dtype in (("f32", np.float32), ("f16", np.float16)):
        A, B, C0 = wl.make_inputs(M, N, K, "uniform", "uniform", seed=10600 + N, c_dtype=dtype)
        got = run_gemm(A, B, C0, mode)
        rows = np.unique([0, M // 3, M // 2, M - 1])
        Cref, S = oracle_mod.gemm_f16(A, B, C0, rows=rows)
        assert_close(got[rows], Cref, S, C0[rows], mode, what=f"{(M, N, K)} {mode}")
