"""Which launches a projection takes (CPU: host arithmetic of the built library): the tile shape, or two side by side, and whether
tiles of two k ranges run as halves."""
import pytest

from tests import host_program


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    exe = host_program.build(tmp_path_factory.mktemp("launches"), "gemm_launches")
    return lambda *row: host_program.run(exe, "%d %d %d %d %d %d\n" % row)[0]


@pytest.mark.parametrize("row, want", [
    # tokens, features, K in 2-byte units, fused q/k/v, SwiGLU, scratch: columns of the first launch, tile rows of either
    ((1409, 11012, 2560, 0, 0, 0), (32, 192, 128)), ((1500, 11012, 2560, 0, 0, 0), (32, 192, 128)), ((3300, 5524, 2560, 0, 0, 0), (14, 192, 128)),
    ((806, 27664, 2560, 0, 1, 0), (51, 192, 256)), ((2000, 13840, 2560, 0, 1, 0), (32, 256, 192)),
    ((1409, 10880, 2560, 1, 0, 0), (32, 192, 128)), ((640, 27648, 5120, 0, 1, 1), (64, 192, 128)),
    ((4447, 11264, 2048, 0, 1, 0), (32, 192, 256)), ((4235, 12288, 1152, 0, 1, 0), (15, 256, 192)),   # short k
    ((385, 11012, 2560, 0, 0, 0), (0, 0, 0)), ((8192, 8192, 8192, 0, 0, 0), (0, 0, 0)), ((1409, 11012, 2568, 0, 0, 0), (0, 0, 0)),
])
def test_columns_of_two_shapes(launches, row, want):
    assert launches(*row)[4:7] == want


@pytest.mark.parametrize("row, halves", [
    ((8061, 5120, 5120, 0, 0, 1), 1), ((6918, 8192, 7168, 0, 0, 1), 1), ((3870, 10240, 8192, 1, 0, 1), 1),   # beside whole tiles
    ((7553, 5120, 13824, 0, 0, 1), 0), ((5648, 4096, 14336, 0, 0, 1), 0),                                      # long k
    ((667, 10240, 8192, 1, 0, 1), 1), ((2854, 2560, 8192, 1, 0, 1), 1),                                        # alone on the chip, and filling it
    ((2406, 2560, 8192, 1, 0, 1), 0), ((2258, 3072, 8192, 0, 0, 1), 0), ((1407, 5120, 13824, 0, 0, 1), 0),     # alone, and not, or of long k
    ((8061, 5120, 5120, 0, 0, 0), 0),                                                                          # nothing is cut without scratch
])
def test_tails_in_halves(launches, row, halves):
    assert launches(*row)[7] == halves


@pytest.mark.parametrize("row, tile", [
    # SwiGLU of at most 256 tokens without scratch, where the shapes' times lie clearly apart (profiles/gemm_whole_tiles.txt)
    ((100, 27648, 2560, 0, 1, 0), (64, 128)), ((130, 14336, 4096, 0, 1, 0), (64, 128)), ((200, 16384, 3072, 0, 1, 0), (64, 128)),
    ((130, 27648, 5120, 0, 1, 0), (128, 256)), ((256, 27648, 5120, 0, 1, 0), (128, 256)), ((264, 27648, 5120, 0, 1, 0), (192, 256)),
])
def test_whole_tiles_of_few_rows(launches, row, tile):
    assert launches(*row)[:2] == tile
