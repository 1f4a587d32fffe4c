"""The split k loop with its parts on different XCDs: counts of workgroups that do not divide by the
number of XCDs, one and several rows of tiles, k tails, a part shorter than the others, and sizes on
either side of the rule's line.  Every tile and part has to be taken exactly once: integers, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2108_13191_amd import binding, workloads as wl   # noqa: E402
from gpu_util import run_gemm                                # noqa: E402


@pytest.mark.parametrize("M,N,K", [
    (17, 464, 3744),        # 4 tiles x 3 parts, fewer workgroups than two rounds of the XCDs
    (35, 312, 3840),        # 3 x 3, one more than there are XCDs
    (151, 344, 9136),       # 2 x 3 tiles x 8 parts, a k tail
    (1100, 136, 5128),      # 9 rows of tiles: two groups of the tile order
    (16, 4200, 8200),       # more than 68 MB, few rows
    (20, 4200, 8200),       # ... and more: 33 tiles, the other order, shifted by a tile from part to part
    (20, 4088, 8712),       # ... 32 tiles: all parts of a tile on one XCD
    (256, 3976, 8200),      # ... and two full tiles of rows
])
def test_every_tile_and_part_once(oracle_mod, M, N, K):
    binding.force_config(-1)
    tiles = -(-M // 128) * -(-N // 128)
    cfg = binding.query_config(False, M, N, K, None, K, None, N, None, N + 8)
    assert cfg["name"] == "w4a_128x128x64" and cfg["grid"] > tiles, cfg
    A, B, _ = wl.make_inputs(M, N, K, "int2", "zeros", seed=M + N, c_dtype=np.float32)
    C0 = np.random.default_rng(K).integers(-4, 5, size=(M, N)).astype(np.float32)
    Cref, _ = oracle_mod.gemm_f16(A, B, C0)
    assert np.array_equal(run_gemm(A, B, C0, "f32", ldc=N + 8), Cref.astype(np.float32))
