"""The forms of the phase-alternating kernel that read and write a large C (96 MB and more, K < 4096) with the
non-temporal hint: every tile form, with and without a k tail, ragged edges, just above and just
below the size, rows of C that begin at 64-byte sectors and that do not.  Integers bit for bit against the oracle on sampled rows."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from gpu_util import config_id, run_gemm
from paper_2108_13191_amd import binding
from paper_2108_13191_amd import workloads as wl

pytestmark = pytest.mark.gpu
CDT = {"f32": np.float32, "f16": np.float16}
P = "pp256x256x64_w2x4_mi16"
NAMES = [P, P + "_chain", P + "_stag", "pp192x256x64_w2x4_mi16", "pp128x256x64_w2x4_mi16", "pp256x192x64_w2x4_mi16", "pp128x128x64_w2x4_mi16"]


@pytest.fixture(autouse=True)
def _unforce():
    yield
    binding.force_config(-1)


@pytest.mark.parametrize("name", NAMES)
@pytest.mark.parametrize("mode", ["f32", "f16"])
def test_large_c(oracle_mod, name, mode):
    binding.force_config(config_id(name))
    # 96.2 MB three times, then 95.9
    for M, N, K, pad in ((5861, 4104, 128, 24), (5861, 4104, 72, 24), (5861, 4104, 72, 0), (5841, 4104, 64, 24)):
        if mode == "f16":
            M *= 2
        A, B, _ = wl.make_inputs(M, N, K, "int2", "zeros", seed=K)
        C0 = ((np.arange(M)[:, None] + np.arange(N)[None, :]) % 9 - 4).astype(CDT[mode])
        got = run_gemm(A, B, C0, mode, ldc=N + pad)
        rows = np.unique(np.concatenate([[0, 1, 127, 128, 255, 256, M - 257, M - 2, M - 1], np.random.default_rng(K).integers(0, M, 40)]))
        Cref, _ = oracle_mod.gemm_f16(A, B, C0, rows=rows)
        want = oracle_mod.round_to_f32(Cref) if mode == "f32" else Cref.astype(np.float16)
        assert np.array_equal(got[rows], want), (name, M, N, K, mode)
