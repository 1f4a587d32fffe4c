"""What runs on few tiles and long k loops, on the sides of the selector's lines where a measurement says so (the
query reports the plan), and results on either side."""
import numpy as np
import pytest

from paper_2108_13191_amd import binding
from paper_2108_13191_amd import workloads as wl


def _name(f16, M, N, K, pad=0):
    return binding.query_config(f16, M, N, K, 16, K + pad, 16, N + pad, 16, N + pad)["name"]


def test_f32_up_to_four_times_as_wide_as_high():
    """B is not wide there: the small tiles are not charged for its latency ((67,96,4104) 6.5 us against 12.0 cut along k,
    from memory 10.4 against 13.8)."""
    for M, N, K, pad in [(67, 96, 4104, 0), (96, 336, 4496, 8), (84, 128, 4608, 64), (107, 240, 4632, 64), (128, 408, 4048, 64),
                       (105, 4712, 2032, 0), (69, 6000, 2024, 0), (82, 5640, 2000, 0)]:           # (... nor at K < 2048)
        assert _name(0, M, N, K, pad).startswith("ks"), (M, N, K)
    # few rows against a wide B stay cut along k
    assert _name(0, 14, 1640, 4976) == "w4a_128x128x64" and _name(0, 3, 1792, 4464) == "w4a_128x128x64"


def test_f16_tiles_of_32_by_32_in_a_second_round():
    """Not where the plan before them is a larger kernel, and not for less than an estimated seventh: (436,2312,5288) 46.2 us on
    128 x 128, 55.2 on 1022 tiles of 32 x 32, (10503,88,3680) 34.0 and 38.3, (290,1616,9736) 42.9 on 64 x 64 tiles, 52.9."""
    for M, N, K, pad in [(436, 2312, 5288, 64), (10503, 88, 3680, 0), (2465, 392, 3400, 0), (10347, 88, 2304, 0), (8238, 72, 3904, 8), (417, 2312, 12480, 0), (340, 2968, 6056, 0)]:
        assert not _name(1, M, N, K, pad).startswith("ks"), (M, N, K)
    for M, N, K, pad in [(290, 1616, 9736, 8), (1763, 264, 3584, 64), (5391, 88, 3200, 0), (196, 2328, 3032, 0)]:
        assert _name(1, M, N, K, pad) == "ks64x64x64_k8", (M, N, K)
    # tall ones up to three quarters of a second round; and one round for an estimated 13 % where it leaves room
    for M, N, K, pad in [(8335, 72, 2080, 0), (8527, 96, 2544, 0), (8213, 88, 3208, 0), (11736, 16, 3376, 0), (9765, 16, 2504, 0), (4330, 96, 3480, 64), (14949, 16, 2592, 0)]:
        assert _name(1, M, N, K, pad) == "ks32x32x64_k8", (M, N, K)
    # two rounds of 32 x 64, and one round of small tiles for a third: as before
    for M, N, K, pad in [(2316, 400, 2392, 0), (2322, 392, 11040, 8), (131, 6376, 12240, 0), (203, 4176, 2184, 64)]:
        assert _name(1, M, N, K, pad) == "ks32x64x64_k8", (M, N, K)
    assert _name(1, 160, 760, 3496).startswith("ks") and _name(1, 10, 1072, 5672) == "ks16x32x64_k8"


def test_f16_nine_rows_of_small_tiles():
    """Rows of 32 x 64 tiles that leave one over the groups of eight that the tile order walks: that row reads all of B alone.
    (272,3584,8128) five stages 46.6 us, small tiles 59.9; (275,3536,13872) 64 x 64 tiling 97.5, 117.  The same against the
    64 x 64 tiling on little more than one of its tiles a compute unit: (137,5448,12688) 86.7, 102.6."""
    for M, N, K, pad in [(272, 3584, 8128, 0), (265, 3584, 3968, 0), (283, 3456, 3136, 0), (265, 3544, 6520, 8)]:
        assert _name(1, M, N, K, pad) == "w4a_128x128x64", (M, N, K)
    for M, N, K, pad in [(275, 3536, 13872, 64), (286, 3304, 14656, 64), (137, 5448, 12688, 0), (156, 5624, 16176, 64), (339, 2816, 11584, 8)]:
        assert _name(1, M, N, K, pad) == "t64x64x64_w2x2", (M, N, K)
    # other counts of rows, more tiles, and against the phase-alternating kernel
    for M, N, K, pad in [(207, 4672, 5504, 0), (323, 2944, 2752, 0), (155, 5824, 15488, 0), (217, 4224, 14480, 0), (468, 2064, 15080, 0), (277, 3344, 6136, 64)]:
        assert _name(1, M, N, K, pad) == "ks32x64x64_k8", (M, N, K)


def test_f32_long_k_loops_with_rows_at_lines():
    """The small tiles' estimates leave out what operands from memory cost there: (205,1984,5504) cut along k 15.3 us, small tiles
    18.0, (3274,64,6144) from memory 18.1 and 22.0, (721,64,6912) 16.0 and 17.5."""
    for M, N, K, pad in [(205, 1984, 5504, 64), (2289, 64, 5632, 0), (3274, 64, 6144, 0), (145, 1472, 6400, 64), (721, 64, 6912, 0), (147, 704, 7744, 64), (173, 2048, 4864, 0)]:
        assert _name(0, M, N, K, pad) == "w4a_128x128x64", (M, N, K)
    # smaller operands up to K = 6200, shorter k loops, clearly better estimates, rows within a line
    for M, N, K, pad in [(136, 960, 5504, 0), (164, 768, 5888, 0), (157, 4736, 3520, 0), (3588, 192, 3584, 0), (5605, 128, 2432, 0), (159, 640, 6336, 0), (3388, 128, 5376, 64), (6495, 64, 5120, 0), (2047, 448, 5248, 0), (1456, 320, 5696, 64), (183, 5376, 4608, 64), (929, 96, 6016, 8), (508, 64, 5056, 0)]:
        assert _name(0, M, N, K, pad).startswith("ks"), (M, N, K)


def _narrow(M, N, K, ldb):
    return binding.query_config(0, M, N, K, 16, K + (-K) % 64, 16, ldb, 16, N)["name"]


def test_f32_up_to_32_columns():
    """Every workgroup of the small tiles reads all of B: where its rows lie on lines of their own (a pitch of 64 and more), and in
    a second round, that pays only up to shorter k loops ((1358,32,8536) at a pitch of 96 cut along k 15.8 us, small tiles 17.3, from
    memory 20.2 and 26.3; (16037,8,5056) at 72 36.5 and 41.1; (13988,32,6784) 39.6 and 43.4)."""
    cut, small = "w4a_128x128x64", "ks"
    for M, N, K, ldb, want in [(1358, 32, 8536, 96, cut), (313, 8, 7368, 72, cut), (6173, 8, 6208, 72, cut), (1465, 16, 5504, 80, small), (614, 16, 6120, 80, small), (5764, 16, 4824, 80, small),
                               (1358, 32, 8536, 32, small), (313, 8, 7368, 8, small),
                               (16037, 8, 5056, 72, cut), (13187, 24, 7408, 88, cut), (14737, 16, 4096, 80, small), (12000, 16, 2176, 80, small),
                               (13988, 32, 6784, 32, cut), (12176, 16, 8448, 16, cut), (14905, 32, 7472, 32, cut), (13339, 8, 6120, 8, small), (13312, 8, 7432, 8, small), (13068, 16, 7344, 16, small), (15488, 8, 8616, 8, small), (14081, 24, 5744, 24, small)]:
        assert _narrow(M, N, K, ldb).startswith(want), (M, N, K, ldb)


def test_f32_two_k_groups():
    """From 23 k steps on and where three calls' matrices fit the last-level cache: (12672,256,2944) 34.4 us, 32.5 on the
    phase-alternating kernel, (12608,256,1280) from memory 22.7 and 21.1."""
    two = "pp128x128x64_w2x2_k2"
    for M, N, K in [(2048, 2048, 2048), (1512, 1536, 1472), (4022, 896, 2944), (2048, 2048, 4096), (335, 8192, 4032), (11712, 192, 3008), (2048, 1920, 1984), (140, 12672, 1664), (256, 11968, 1920), (428, 6848, 5248), (9536, 320, 5888)]:
        assert _name(0, M, N, K) == two, (M, N, K)
    for M, N, K in [(12608, 256, 1280), (2048, 2048, 1408), (12672, 256, 2944), (133, 11776, 4736), (180, 16000, 5504), (150, 13440, 5184), (134, 15744, 1536), (256, 16000, 1664)]:
        assert _name(0, M, N, K) == "pp128x128x64_w2x4_mi16", (M, N, K)


def test_any_alignment_little_more_than_a_round_of_256_by_256():
    """Rows at 8-byte addresses and better cost the 128 x 128 form no lane a clock: (2840,6261,3235) at pitches of 3264 and 6262 165 us on it,
    182 on 300 workgroups of 256 x 256."""
    def name(f16, M, N, K, lda, ldb, a=16, b=16):
        return binding.query_config(f16, M, N, K, a, lda, b, ldb, 16, N + 1)["name"]
    large, small = "generic256x256x64", "generic128x128x64"
    assert name(0, 2840, 6261, 3235, 3264, 6262) == small and name(1, 2971, 6185, 3640, 3648, 6188) == small and name(0, 4125, 4199, 2854, 2854, 4224) == small
    assert name(0, 2840, 6261, 3235, 3235, 6261) == large                       # odd rows
    assert name(0, 2840, 6261, 3235, 3264, 6262, a=18) == large                 # odd rows: where they begin counts too
    assert name(0, 3260, 6055, 8565, 8568, 6056) == large                       # clearly estimated faster
    assert name(0, 10925, 1975, 7443, 7448, 1980) == large                      # more than a quarter of a second round


@pytest.mark.gpu
def test_results_on_both_sides(oracle_mod):
    """One problem on either side of each line, on the GPU: sampled rows against the oracle."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from gpu_util import assert_close, run_gemm
    for mode, M, N, K, pad in [("f32", 67, 96, 4104, 0), ("f32", 14, 1640, 4976, 0), ("f16", 436, 2312, 5288, 64), ("f16", 2316, 400, 2392, 0), ("f16", 290, 1616, 2056, 8),
                               ("f16", 272, 3584, 2112, 0), ("f16", 323, 2944, 2752, 0), ("f32", 205, 1984, 5504, 64), ("f32", 164, 768, 5888, 0), ("f32", 1358, 32, 8536, 64),
                               ("f32", 13339, 8, 6120, 0), ("f32", 1512, 1536, 1472, 0), ("f32", 1512, 1536, 1408, 0), ("f32", 2840, 6261, 449, 29), ("f16", 2840, 6261, 449, 0)]:
        dtype = {"f32": np.float32, "f16": np.float16}[mode]
        A, B, C0 = wl.make_inputs(M, N, K, "normal_rsqrtk", "uniform", seed=10700 + N, c_dtype=dtype)
        got = run_gemm(A, B, C0, mode, lda=K + pad, ldb=N + pad)
        rows = np.unique([0, M // 3, M // 2, M - 1])
        Cref, S = oracle_mod.gemm_f16(A, B, C0, rows=rows)
        assert_close(got[rows], Cref, S, C0[rows], mode, what=f"{(M, N, K)} {mode}")
