"""Which tile form automatic selection takes where the estimates of launch_cost are corrected by measured lines."""
import pytest

from paper_2108_13191_amd import binding

P = "pp128x128x64_w2x4_mi16"


@pytest.fixture(autouse=True)
def _unforce():
    binding.force_config(-1)


def name(f16, M, N, K):
    return binding.query_config(f16, M, N, K, 256, K, 256, N, 256, N)["name"]


@pytest.mark.parametrize("f16", [0, 1])
def test_one_round_of_128x256_in_place_of_shared_128x128(f16):
    wide = "pp128x256x64_w2x4_mi16"
    assert name(f16, 2560, 2560, 960) == wide and name(f16, 2560, 2560, 952) == P            # 400 tiles, 200; 15 k steps
    assert name(f16, 2048, 2176, 1088) == wide and name(f16, 2048, 2176, 1080) == P          # 272, 144; 17
    assert name(f16, 4096, 2048, 1536) == wide                                              # 512 and 256
    assert name(f16, 4096, 2056, 1536) != wide                                              # 288 of 128 x 256
    assert name(f16, 2304, 1800, 2048) == wide and name(f16, 2048, 1920, 1280) != wide      # 270 of 128 x 128, and 240


@pytest.mark.parametrize("f16", [0, 1])
def test_two_short_rounds_of_128x128_in_place_of_192x256(f16):
    tall = "pp192x256x64_w2x4_mi16"
    assert name(f16, 4224, 4352, 400) == P                                                  # 33 x 34 = 1122 tiles of 128 x 128, two rounds are 1024, 2.2 are 1126
    assert name(f16, 4224, 4352, 408) == tall
    assert name(f16, 4224, 4480, 304) == P and name(f16, 4224, 4480, 312) == tall           # 1155


@pytest.mark.parametrize("f16", [0, 1])
def test_one_short_launch_in_place_of_two(f16):
    last = 184
    def q(M, N, K):
        return binding.query_config(f16, M, N, K, 256, K, 256, N, 256, N)
    for M, N in ((15859, 1616), (7200, 3632), (4962, 5312)):                                # 1612, 1653 and 1638 tiles: up to 3.3 rounds
        assert q(M, N, last)["name"] == P and q(M, N, last)["split_rows"] == 0
    assert q(8700, 3632, last)["name"] != P                                                 # 1972
    for M, N in ((3138, 6272), (407, 35264), (2559, 7680), (1777, 13056)):                  # 1225, 1104, 1200 and 1428: longer loops up to three rounds
        for K in (192, 272, 328):
            assert q(M, N, K)["name"] == P and q(M, N, K)["split_rows"] == 0, (M, N, K)
        assert q(M, N, 336)["split_rows"] > 0


def test_two_k_groups_in_the_f16_mode():
    two = "pp128x128x64_w2x2_k2"
    assert name(1, 2048, 1280, 832) == two and name(1, 2048, 1280, 768) == P                # 160 tiles; 13 k steps
    assert name(1, 2048, 1280, 1984) == two and name(1, 2048, 1280, 2048) == "w4a_128x128x64"
    assert binding.query_config(1, 2048, 1280, 3000, 256, 3008, 256, 1280, 256, 1280)["name"] == two        # a k tail
    assert binding.query_config(1, 2048, 1280, 1024, 256, 1032, 256, 1280, 256, 1280)["name"] == P          # rows that begin within a line
    assert name(1, 256, 16384, 1280) == two and name(1, 256, 16384, 1408) == P              # 55 MB
    assert name(1, 2048, 1024, 960) == two and name(1, 2048, 1024, 640) == P                # half a chip of tiles: 11 k steps
    assert name(1, 2048, 1024, 1024) == "w4a_128x128x64"
    assert name(1, 1024, 896, 960) != two                                                   # 56 tiles


def test_small_tiles_keep_their_problems_from_two_k_groups():
    """f16, 66 to 77 tiles of 128 x 128: 32 x 64 tiles, which had them and are faster there in every use."""
    for M, N, K in ((195, 4160, 896), (81, 9152, 960), (86, 9408, 960), (88, 9088, 896)):
        assert name(1, M, N, K) == "ks32x64x64_k8"


def test_two_k_groups_for_left_over_rows():
    """The second of two launches: in the f16 mode as where the tiles are all there is."""
    for f16, M, N, K in ((1, 3163, 6400, 1024), (1, 5120, 4096, 832), (1, 2539, 7360, 1472), (0, 2539, 7360, 1472)):
        q = binding.query_config(f16, M, N, K, 256, K, 256, N, 256, N)
        assert q["split_rows"] > 0 and binding.describe_config(q["id2"])["name"] == "pp128x128x64_w2x2_k2"
