"""The forms of the phase-alternating kernel that read and write a large C (300 MB and more, 256 <= K < 4096) with the
non-temporal hint: every tile form, with and without a k tail, ragged edges, just above and just
below the size, rows of C that begin at 64-byte sectors and that do not.  Integers bit for bit against the oracle on sampled rows."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from gpu_util import DevMat, config_id
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
    # 300.0 MB three times (the third at rows within a sector), then 299.4
    for M, N, K, pad in ((9147, 8200, 320, 24), (9147, 8200, 264, 24), (9147, 8200, 264, 0), (9127, 8200, 256, 24)):
        if mode == "f16":
            M *= 2
        A, B, _ = wl.make_inputs(M, N, K, "int2", "zeros", seed=K)
        rows = np.unique(np.concatenate([[0, 1, 127, 128, 255, 256, M - 257, M - 2, M - 1], np.random.default_rng(K).integers(0, M, 40)]))
        C0 = ((rows[:, None] + np.arange(N)[None, :]) % 9 - 4).astype(CDT[mode])
        dA, dB = DevMat(A, nan_canary=True), DevMat(B, nan_canary=True)
        buf = torch.full((M + 1, N + pad), -1234.0, dtype=torch.float32 if mode == "f32" else torch.float16, device="cuda")
        C = buf[:M, :N]
        C.copy_((torch.arange(M, device="cuda", dtype=torch.int16)[:, None] % 9 + torch.arange(N, device="cuda", dtype=torch.int16)[None, :]) % 9 - 4)
        fn = binding.gemm_f16_f32acc if mode == "f32" else binding.gemm_f16_f16acc
        binding.check(fn(M, N, K, dA.ptr, dA.ld, dB.ptr, dB.ld, buf, N + pad, torch.cuda.current_stream().cuda_stream))
        got = C[torch.from_numpy(rows).cuda()].cpu().numpy()
        assert bool((buf[M] == -1234.0).all()) and bool((buf[:, N:] == -1234.0).all()), "memory outside C was written"
        Cref, _ = oracle_mod.gemm_f16(A[rows], B, C0)
        want = oracle_mod.round_to_f32(Cref) if mode == "f32" else Cref.astype(np.float16)
        assert np.array_equal(got, want), (name, M, N, K, mode)
