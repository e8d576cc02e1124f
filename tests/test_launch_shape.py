"""The launch rules of csrc/launch.h, compiled for the host (tests/native/launch_rules.cpp):
the order in which blocks take tiles, a permutation of the grid for every run and grid size
with each XCD's blocks in stretches of `run` neighbours inside the whole groups; and the
tiles that a call is cut into."""
import os
import subprocess

import pytest

XCDS = 8


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    exe = tmp_path_factory.mktemp("launch_rules") / "launch_rules"
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(root, "paper_2609_18178_amd", "csrc"), "-o", str(exe),
                    os.path.join(root, "tests", "native", "launch_rules.cpp")], check=True)
    return lambda *args: subprocess.run([str(exe), *map(str, args)], capture_output=True, text=True,
                                        check=True).stdout.split()


@pytest.mark.parametrize("run", [16, 32, 128])
@pytest.mark.parametrize("grid", [1, 7, 8, 127, 128, 129, 255, 256, 257, 1023, 1024, 1025, 2048, 2500, 32768, 40001])
def test_every_tile_is_taken_once(rules, grid, run):
    tiles = [int(x) for x in rules("dealt", grid, run)]
    assert sorted(tiles) == list(range(grid))
    for first in range(0, grid - XCDS * run + 1, XCDS * run):
        for xcd in range(XCDS):
            mine = [tiles[b] for b in range(first + xcd, first + XCDS * run, XCDS)]
            assert mine == list(range(first + xcd * run, first + (xcd + 1) * run))


@pytest.mark.parametrize("mode", range(7))
@pytest.mark.parametrize("elems", [1, 100_003, 1 << 20, 3 << 20, 16 << 20, 453_001_472])
def test_calls_without_a_workspace_take_long_tiles(rules, mode, elems):
    """Each tile of such a call adds to the same word, so it has at least 4096 elements."""
    assert int(rules("tile", mode, elems, elems, 0)[0]) >= 4096
    assert int(rules("tile", mode, elems, elems, 1)[0]) in (1024, 4096)


@pytest.mark.parametrize("mode", [0, 3])
def test_commits_of_the_longest_segments_fit_a_launch(rules, mode):
    """A segment of up to 2^24 - 1 tiles of 4096 elements fits one launch, also where its
    usual tiles, of 1024, would not."""
    most = 2 ** 24 - 1
    assert int(rules("tile", mode, most * 1024 - 1, most * 1024 - 1, 1)[0]) == 1024
    assert int(rules("tile", mode, most * 2048, most * 1024 - 1, 1)[0]) == 1024  # several segments: several launches
    for longest in (most * 1024 + 1, 2 ** 24 * 1024, most * 4096):
        elems = int(rules("tile", mode, longest, longest, 1)[0])
        assert -(-longest // elems) <= most
