"""The heights of row tiles that launches are cut into: never more than the kernels that run them have code for, and what they are at some sizes."""
import ctypes

import pytest

import paper_2106_10715_amd as M
from tile_rows import N_CU, heights, lib


def _in_range(T, d, f, E, k, gather, e_count, rows):
    cfg, out = M.MoeCfg.make(T, d, f, E, k, "bf16"), (ctypes.c_int * 3)()
    at, rule = ctypes.addressof(cfg), lib().tile_rows
    most, most_down, least = lib().most_rows(gather), lib().most_rows(0), lib().least_rows()
    for n in rows:
        rule(at, gather, N_CU, e_count, n, out)
        assert least <= out[0] <= most and least <= out[1] <= most_down and out[0] % 16 == 0 and out[1] % 16 == 0, (n, *out)


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


# The heights on 256 compute units, where another choice has cost (layer us, another one / this): few items in the up-projection and none missing in the
# down-projection, 248 / 175, 381 / 326, 125 / 98; experts around a limit, 523 / 413, 539 / 463; items for less than 0.8 of the units, 48 / 40 with an uneven load;
# calls whose tests count on a list for each product; and calls that have always been cut like this.
@pytest.mark.parametrize("T,d,f,E,k,want", [
    (6400, 4096, 256, 64, 1, (96, 224, False)), (22400, 4096, 192, 32, 1, (256, 288, False)), (12800, 1024, 256, 64, 1, (160, 320, True)),
    (1300, 4096, 10240, 4, 1, (256, 96, False)), (2535, 1984, 5376, 8, 3, (320, 288, False)), (6000, 1024, 2048, 12, 1, (256, 128, False)),
    (2000, 512, 1024, 4, 1, (96, 64, False)), (1010, 256, 1536, 3, 1, (96, 64, False)), (2043, 1024, 1536, 8, 1, (128, 64, False)),
    (466, 1024, 320, 12, 1, (64, 64, True)), (400, 512, 1024, 4, 1, (64, 64, True)), (2048, 4096, 10240, 8, 1, (320, 160, False)), (65536, 4096, 10240, 32, 1, (272, 272, False)),
    (4096, 4096, 10240, 32, 1, (224, 224, False)), (512, 4096, 10240, 32, 1, (224, 224, False)), (40, 4096, 10240, 32, 1, (64, 64, False))])
def test_heights(T, d, f, E, k, want):
    assert heights(T, d, f, E, k, gather=T * k // E <= 160) == want
