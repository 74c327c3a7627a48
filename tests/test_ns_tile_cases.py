"""The sizes that the GPU tests of the Newton-Schulz products use run the output tiles that the tests
say they run, and between them every tile in every form (no GPU needed)."""
from helpers import ns_tiles
from test_gpu_inner_step import SIDE_BY_SIDE, SMALL_TILE_UPDATES
from test_gpu_newton_schulz import MANY_TILES, RING, SAME_BITS


def test_cases_run_the_tiles_they_name():
    for c, m, n, tiles in MANY_TILES + RING:
        assert ns_tiles([(c, m, n)]) == [tiles], (c, m, n)
    for m, n, counts in SAME_BITS:
        for c, tiles in counts.items():
            assert ns_tiles([(c, m, n)]) == [tiles], (c, m, n)
    for shapes, tiles in SIDE_BY_SIDE + SMALL_TILE_UPDATES:
        assert ns_tiles(shapes) == tiles, shapes


def test_every_tile_is_covered():
    seen = {(form, tile, m > n) for _, m, n, tiles in MANY_TILES + RING for form, tile in enumerate(tiles)}
    for tile in (64, 128, 256):
        assert {(0, tile, False), (0, tile, True), (1, tile, False), (2, tile, False), (2, tile, True)} <= seen, tile
    # weights updated by the last product of a tall matrix, from the smallest tile up
    assert any(tile[2] == 64 and m > n for shapes, tiles in SMALL_TILE_UPDATES for (_, m, n), tile in zip(shapes, tiles))


def test_short_products_never_take_the_64_tile():
    for count in (1, 7, 60, 500):
        for long_side in (640, 1024, 8192):
            for shape in ((128, long_side), (long_side, 128)):
                gram, poly, apply = ns_tiles([(count, *shape)])[0]
                assert poly == apply == 128          # K = 128: the 64 tile's ring needs 256
