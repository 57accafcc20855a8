"""The k ranges a projection's sums are cut into (CPU: host arithmetic of the built library).

Which tiles split their k range fixes the order of every sum.  It depends on the sizes alone -- not on the operands' width,
not on the tile shape that happens to be fastest -- and the sizes below pin it: a row that changes reorders sums that
serving results were recorded with."""
import pytest

from tests import host_program

WHOLE = None

# (tokens, features, K in 2-byte units, fused q/k/v epilogue, SwiGLU): (tile rows, tile features, split tiles, ways), or WHOLE
CUTS = {
    (257, 2560, 4096, 1, 0): (192, 256, 20, 5), (257, 3584, 5120, 1, 0): (192, 256, 28, 5),
    (300, 7168, 2560, 1, 0): (192, 256, 56, 2), (300, 7168, 5120, 1, 0): (192, 256, 56, 3),
    (300, 8192, 3584, 0, 0): (192, 256, 64, 3), (300, 8192, 4096, 0, 0): (192, 256, 64, 3),
    (384, 5120, 2560, 0, 0): (192, 256, 40, 3), (385, 3584, 5120, 1, 0): (128, 256, 56, 4),
    (512, 5120, 6912, 0, 0): (192, 256, 60, 4), (512, 8192, 14336, 0, 0): (256, 256, 64, 4),
    (640, 10240, 8192, 1, 0): (256, 256, 120, 2), (769, 3584, 5120, 1, 0): (192, 256, 70, 3),
    (769, 5120, 27648, 0, 0): (256, 256, 80, 3), (1000, 57344, 4096, 0, 1): (256, 256, 128, 2),
    (1152, 2560, 4096, 1, 0): (192, 256, 60, 3), (3001, 2560, 8192, 1, 0): (256, 256, 120, 2),
    # the projections of a 13B layer at 640 tokens (128 decode rows and a 512-token chunk), 16-bit and 8-bit
    (640, 15360, 5120, 1, 0): WHOLE, (640, 15360, 2560, 1, 0): WHOLE, (640, 27648, 5120, 0, 1): WHOLE, (640, 27648, 2560, 0, 1): WHOLE,
    (384, 15360, 2560, 1, 0): WHOLE, (384, 55296, 5120, 0, 1): WHOLE, (512, 15360, 5120, 1, 0): WHOLE,
    (769, 5120, 2560, 0, 0): WHOLE, (1152, 8192, 4096, 0, 0): WHOLE, (2048, 8192, 8192, 0, 0): WHOLE,
    (2048, 57344, 8192, 0, 1): WHOLE, (2304, 7168, 2560, 1, 0): WHOLE, (3001, 3584, 2560, 1, 0): WHOLE,
}


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    exe = host_program.build(tmp_path_factory.mktemp("plans"), "gemm_plans")
    return lambda rows: host_program.run(exe, "".join("%d %d %d %d %d\n" % row for row in rows))


def test_cuts_are_pinned(plans):
    rows = list(CUTS)
    for row, got in zip(rows, plans(rows)):
        want = CUTS[row]
        assert (got[2:] == (0, 1)) if want is WHOLE else (got == want), (row, got, want)


@pytest.mark.parametrize("row,tile", [
    ((580, 27648, 5120, 0, 1), (192, 256)), ((640, 27648, 5120, 0, 1), (192, 256)), ((640, 27648, 2560, 0, 1), (192, 256)),
    ((600, 55296, 5120, 0, 1), (256, 256)), ((300, 57344, 8192, 0, 1), (192, 256)), ((3000, 1408, 256, 0, 1), (64, 128)),
    ((2500, 2816, 512, 0, 1), (128, 128)), ((1152, 5120, 5120, 0, 0), (128, 256)), ((1280, 5120, 5120, 0, 0), (128, 256)),
    ((512, 15360, 5120, 1, 0), (128, 256)), ((4200, 15360, 5120, 1, 0), (256, 256)), ((806, 7168, 2560, 1, 0), (128, 256)),
])
def test_whole_tiles_take_the_measured_fastest_shape(plans, row, tile):
    """Sizes where the measured times of the shapes lie clearly apart (profiles/gemm_whole_tiles.txt)."""
    assert plans([row]) == [(*tile, 0, 1)]
