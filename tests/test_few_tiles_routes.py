"""What runs on few tiles and long k loops, on the sides of the selector's lines where a measurement says so (no launch: the
query reports the plan)."""
from paper_2108_13191_amd import binding


def _name(f16, M, N, K, pad=0):
    return binding.query_config(f16, M, N, K, 16, K + pad, 16, N + pad, 16, N + pad)["name"]


def test_f32_up_to_four_times_as_wide_as_high():
    """B is not wide there: the small tiles are not charged for its latency ((67,96,4104) 6.5 us against 12.0 cut along k,
    from memory 10.4 against 13.8)."""
    for M, N, K, pad in [(67, 96, 4104, 0), (96, 336, 4496, 8), (84, 128, 4608, 64), (107, 240, 4632, 64), (128, 408, 4048, 64)]:
        assert _name(0, M, N, K, pad).startswith("ks"), (M, N, K)
    # few rows against a wide B stay cut along k
    assert _name(0, 14, 1640, 4976) == "w4a_128x128x64" and _name(0, 3, 1792, 4464) == "w4a_128x128x64"
