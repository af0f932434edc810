"""The choice between the streaming GEMM kernel and the LDS-tiled variants (host code only) against measured times."""
import pytest

# (M, K, N, epilogue, activation), microseconds: streaming kernel, then the variants 0 .. 4 of spec_gemm_tile_variant.
# Medium and few rows, where a launch has one or two rounds; products whose tiles the XCDs share out unevenly among them
# (4128 x 3840: 255 tiles of 256 x 256, of which one XCD gets 36), and large ones.
MEASURED = [
    ((3366, 1024, 4096, 0, 1), (50.4, 53.2, 51.0, 46.2, 65.6, 63.9)),
    ((1500, 4096, 1024, 2, 0), (34.0, 88.8, 47.0, 41.2, 42.0, 34.4)),
    ((3366, 4096, 1024, 2, 0), (60.6, 90.1, 48.8, 43.4, 44.2, 38.2)),
    ((4128, 1280, 3840, 0, 0), (67.0, 80.4, 49.9, 57.6, 62.4, 72.3)),
    ((1100, 5120, 1280, 2, 0), (38.9, 110.5, 60.4, 51.6, 52.2, 42.5)),
    ((3100, 5120, 1280, 2, 0), (75.8, 110.9, 61.8, 69.0, 57.4, 85.9)),
    ((3100, 1280, 1280, 0, 2), (23.4, 46.4, 23.1, 22.9, 22.5, 30.9)),
    ((2304, 1280, 1280, 3, 0), (32.9, 43.0, 22.2, 19.9, 21.6, 18.6)),
    ((256, 1280, 33280, 1, 0), (45.1, 48.2, 58.4, 51.8, 66.0, 57.2)),
    ((330, 5120, 7168, 0, 0), (43.9, 110.6, 73.8, 67.2, 62.3, 53.0)),
    ((576, 5120, 7168, 0, 0), (59.0, 112.6, 75.6, 71.0, 66.1, 90.7)),
    ((2100, 5120, 7168, 0, 0), (184.2, 237.8, 174.4, 160.5, 190.5, 206.5)),
    ((2304, 5120, 7168, 0, 0), (187.4, 241.5, 183.7, 168.3, 194.6, 215.4)),
    ((6144, 5120, 7168, 0, 0), (500.2, 428.2, 440.1, 476.4, 489.5, 582.3)),
    ((576, 5120, 5120, 2, 0), (48.6, 113.1, 75.3, 67.8, 64.2, 53.1)),
    ((3100, 5120, 27648, 4, 0), (890.3, 863.1, 943.5, 962.7, 1055.3, 1142.3)),
    ((6144, 5120, 27648, 4, 0), (1717.9, 1596.7, 1906.1, 1908.1, 2095.0, 2187.2)),
    ((576, 13824, 5120, 2, 0), (104.4, 287.6, 194.6, 175.0, 160.9, 133.5)),
    ((405, 2048, 11264, 4, 0), (68.4, 54.6, 42.0, 32.8, 48.0, 43.7)),
    ((720, 8192, 4096, 0, 0), (65.7, 182.3, 109.7, 101.5, 90.6, 77.9)),
]


@pytest.mark.parametrize("shape,us", MEASURED)
def test_chosen_kernel_is_not_behind(lib, shape, us):
    """Runs of one product differ by up to 3 %: no more than 4 % behind the streaming kernel, 12 % behind the best."""
    v = lib.lib.spec_gemm_tile_variant(*shape)
    assert us[v + 1] <= 1.04 * us[0] and us[v + 1] <= 1.12 * min(us), (v, us)


def test_what_the_tiles_cannot_take(lib):
    f = lib.lib.spec_gemm_tile_variant
    assert f(255, 1024, 4096, 0, 0) == -1 and f(4096, 960, 4096, 0, 0) == -1 and f(4096, 1088, 4096, 0, 0) == -1
    assert f(4096, 1024, 4064, 4, 0) == -1 and f(4096, 1024, 4065, 0, 0) == -1 and f(0, 1024, 4096, 0, 0) == -1
    assert f(4096, 1152, 4096, 0, 0) in (0, 1, 2)          # four stages need a K of whole 256s
    assert f(300, 1024, 1024, 2, 0) == -1                  # the narrow-tile kernel's
