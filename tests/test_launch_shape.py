"""The order in which blocks take tiles (dealt_tile in kernels.hip, in Python):
a permutation of the grid for every run and grid size, with each XCD's blocks in
stretches of `run` neighbours inside the whole groups."""
import pytest

XCDS = 8


def dealt(block, grid, run):
    group = XCDS * run
    r = block % group
    first = block - r
    return first + r % XCDS * run + r // XCDS if grid - first >= group else block


@pytest.mark.parametrize("run", [16, 32, 128])
@pytest.mark.parametrize("grid", [1, 7, 8, 127, 128, 129, 255, 256, 257, 1023, 1024, 1025, 2048, 2500, 32768, 40001])
def test_every_tile_is_taken_once(grid, run):
    tiles = [dealt(b, grid, run) for b in range(grid)]
    assert sorted(tiles) == list(range(grid))
    for first in range(0, grid - XCDS * run + 1, XCDS * run):
        for xcd in range(XCDS):
            mine = [tiles[b] for b in range(first + xcd, first + XCDS * run, XCDS)]
            assert mine == list(range(first + xcd * run, first + (xcd + 1) * run))
