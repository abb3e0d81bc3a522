"""The heights of row tiles that launches are cut into: never more than the kernels that run them have code for, and what they are at some sizes."""
import ctypes

import pytest

import paper_2106_10715_amd as M
from tile_rows import N_CU, heights, lib


def _in_range(T, d, f, E, k, gather, e_count, rows):
    cfg = M.MoeCfg.make(T, d, f, E, k, "bf16")
    at, up_rows, down_rows = ctypes.addressof(cfg), lib().tile_rows_up, lib().tile_rows_down
    most, most_down, least = lib().most_rows(gather), lib().most_rows(0), lib().least_rows()
    for n in rows:
        up = up_rows(at, gather, N_CU, e_count, n)
        down = down_rows(at, e_count, n, up, N_CU)
        assert least <= up <= most and least <= down <= most_down and up % 16 == 0 and down % 16 == 0, (n, up, down)


# Streamed layers launch every expert alone, whatever the mean of the layer, and look its rows up in x up to a mean of 160.
@pytest.mark.parametrize("T,k,E", [(1280, 1, 8), (2000, 1, 16), (2560, 1, 16), (1280, 2, 16), (5120, 1, 32), (40000, 1, 256)])
@pytest.mark.parametrize("d,f", [(256, 10240), (4096, 10240), (1024, 4096), (64, 64), (320, 512), (4096, 448)])
@pytest.mark.parametrize("gather", [0, 1])
def test_single_experts_of_a_layer(T, k, E, d, f, gather):
    _in_range(T, d, f, E, k, gather, 1, range(1, T * k + 1))


@pytest.mark.parametrize("E", [1, 4, 12, 33, 64, 256])
@pytest.mark.parametrize("d,f", [(4096, 10240), (1024, 2048), (64, 64), (320, 512), (4096, 448), (64, 10240)])
@pytest.mark.parametrize("gather", [0, 1])
def test_whole_layers(E, d, f, gather):
    for mean in (*range(1, 200, 7), *range(200, 700, 11), 1000, 2000, 5000, 100000):
        T = E * mean + E // 2
        if T * max(d, f) < 2 ** 31:
            _in_range(T, d, f, E, 1, gather, E, [T])
