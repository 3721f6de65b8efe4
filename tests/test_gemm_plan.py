"""Which kernel the cost rule of the matrix product gives to the sizes that the GPU tests of the tiles run: a change of
its constants must not drop a kernel from those tests unnoticed."""
import pytest

from paper_2201_05500_amd.binding_mlp import ctr_debug_mlp_gemm_plan as plan
from tests.test_gpu_gemm_tiles import BITS, SIZES

ROOM = 32 << 20  # the scratch those tests give


def test_sizes_cover_every_tile_split_and_not():
    taken = {(tile, items > 1, ranges > 1) for tile, items, ranges, _ in
             [plan(*s, ROOM) for s in SIZES + BITS] + [plan(*s, 0) for s in SIZES + BITS]}
    assert {(64, False, False), (64, False, True), (64, True, True), (128, False, False), (128, True, True),
            (256, False, False), (256, True, True)} <= taken


def test_ranges_of_the_sizes_compared_bit_by_bit():
    lengths = {s: plan(*s, ROOM)[2:] for s in BITS}
    assert lengths == {(72, 136, 264): (1, 320), (640, 96, 640): (3, 256), (264, 200, 1288): (6, 256),
                       (136, 72, 9224): (29, 320), (1000, 400, 5768): (19, 320), (1032, 520, 5768): (13, 448),
                       (1032, 520, 8200): (15, 576), (16, 200, 2160): (9, 256), (16, 200, 2560): (10, 256)}
    for (m, n, k), (ranges, length) in lengths.items():
        assert length % 64 == 0 and (ranges - 1) * length < k <= ranges * length
        assert plan(m, n, k, 0)[2] == 1                      # no room for partial sums: one range


@pytest.mark.parametrize("size,tile,split", [((176, 24, 848), 64, True), ((8, 8, 960), 64, True), ((64, 64, 512), 64, False),
                                             ((14584, 600, 8), 256, False), ((7384, 464, 8), 128, False), ((2000, 400, 8), 64, False)])
def test_lines_between_tiles_and_splits(size, tile, split):
    """Contractions of 13 steps and more are split where the chip has room; large outputs of short ones take larger tiles."""
    got, items, _, _ = plan(*size, ROOM)
    assert (got, items > 1) == (tile, split)


@pytest.mark.parametrize("bad", [(0, 8, 8), (8, 12, 8), (8, 8, 4)])
def test_refused_sizes(bad):
    with pytest.raises(ValueError):
        plan(*bad, 0)
