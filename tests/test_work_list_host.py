"""The work list of the expert FFN kernels, compiled for the CPU: every row of every expert in exactly one tile, at every size the
argument checks let through (T k max(d, f) < 2^31, so up to 2^25 rows)."""
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("work_list") / "work_list")
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2106_10715_amd", "csrc"), os.path.join(HERE, "work_list_host.cpp"), "-o", exe, "-lpthread"], check=True)

    def tiles_of(offsets, tile_m, total):
        line = " ".join(map(str, [len(offsets) - 1, tile_m, total, total // 64 + len(offsets) - 1, *offsets]))
        out = subprocess.run([exe], input=line, capture_output=True, text=True, check=True, timeout=60).stdout
        return np.array(out.split(), dtype=np.int64)[1:].reshape(-1, 4)

    def run(counts, tile_m):
        offsets = np.concatenate([[0], np.cumsum(counts)])
        return tiles_of(offsets, tile_m, int(offsets[-1])), offsets
    run.tiles_of = tiles_of
    return run


def check(tiles, offsets, tile_m):
    counts = np.diff(offsets)
    assert tiles[:, 2].min() >= 1 and tiles[:, 2].max() <= tile_m
    by_row = tiles[np.argsort(tiles[:, 1])]
    assert by_row[0, 1] == 0 and np.array_equal(by_row[1:, 1], (by_row[:, 1] + by_row[:, 2])[:-1])     # one after the other, no gap
    assert by_row[-1, 1] + by_row[-1, 2] == offsets[-1]
    assert (tiles[:, 1] >= offsets[tiles[:, 0]]).all() and (tiles[:, 1] + tiles[:, 2] <= offsets[tiles[:, 0] + 1]).all()
    assert ((tiles[:, 1] - offsets[tiles[:, 0]]) % 16 == 0).all()
    assert np.array_equal(np.bincount(tiles[:, 0], minlength=len(counts)), -(-counts // tile_m))
    assert np.array_equal(tiles[:, 3], (-(-counts // tile_m))[tiles[:, 0]])


@pytest.mark.parametrize("counts,tile_m", [
    ([2965819], 256), ([2965820], 256), ([3000000], 256), ([2 ** 25 - 1], 256),       # around the first 32-bit overflow of tile x blocks, the largest
    ([3000000], 64), ([2 ** 25 - 1], 64), ([2595100], 224), ([2 ** 25 - 1], 320),       # other tile heights
    ([5, 3000000, 0, 100], 256), ([16 * 2 ** 20 - 3, 700, 16 * 2 ** 20 + 1], 192),    # and among small experts
])
def test_large_experts(plan, counts, tile_m):
    tiles, offsets = plan(counts, tile_m)
    check(tiles, offsets, tile_m)


@pytest.mark.parametrize("tile_m", [64, 96, 224, 256, 288, 320])
@pytest.mark.parametrize("E,mean,skew", [(1, 40, 0), (1, 5000, 0), (7, 100, 1), (7, 400, 2), (33, 230, 1), (256, 3, 1), (256, 300, 3)])
def test_rows_once(plan, E, mean, skew, tile_m):
    rng = np.random.default_rng(E + mean + tile_m)
    share = rng.random(E) ** (1 + 2 * skew)
    counts = np.floor(share / share.sum() * E * mean).astype(int) + 1
    tiles, offsets = plan(counts, tile_m)
    check(tiles, offsets, tile_m)


def test_order(plan):
    """Few rows per expert: the highest tiles first.  Many: groups of four tiles of experts with several among groups of four of the others."""
    tiles, _ = plan([100, 30, 256, 80, 0, 250], 256)
    assert tiles[:, 0].tolist() == [2, 5, 0, 3, 1]
    tiles, _ = plan([2000] * 2 + [200] * 8, 256)
    several = (tiles[:, 3] > 1).reshape(-1, 4)
    assert (several.all(1) | ~several.any(1)).all() and 0 < (np.diff(several[:, 0].astype(int)) != 0).sum() >= 3


@pytest.mark.parametrize("offsets", [[-5, 2 ** 31 - 1, -2 ** 31, 7], [0, 33000000, 0, 33000000], [33000000, -2 ** 31, 2 ** 31 - 1, -1]])
def test_offsets_out_of_range(plan, offsets):
    """Whatever the offsets hold, no tile reaches outside the rows."""
    tiles = plan.tiles_of(offsets, 64, 33000000)
    assert tiles.size == 0 or (tiles[:, 1].min() >= 0 and tiles[:, 2].min() >= 1 and tiles[:, 2].max() <= 64 and (tiles[:, 1] + tiles[:, 2]).max() <= 33000000)
