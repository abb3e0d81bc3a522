"""The library's rules for the heights of row tiles (ffn_tiles.h), compiled for the CPU: what a launch cuts its rows into."""
import ctypes
import functools
import os
import subprocess
import tempfile

import paper_2106_10715_amd as M

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
N_CU = 256


@functools.lru_cache(maxsize=None)
def lib():
    with tempfile.TemporaryDirectory() as tmp:
        so = os.path.join(tmp, "tile_rows.so")
        subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", os.path.join(ROOT, "include"),
                        "-I", os.path.join(ROOT, "paper_2106_10715_amd", "csrc"), os.path.join(HERE, "tile_rows_host.cpp"), "-o", so], check=True)
        rules = ctypes.CDLL(so)
    rules.tile_rows.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_long, ctypes.c_void_p]
    rules.few_rows_layer.argtypes = [ctypes.c_void_p, ctypes.c_int]
    return rules


def heights(T, d, f, E, k=1, gather=False, e_count=None, max_rows=None):
    """(up, down, narrow): most rows of a tile of the two kernels in a launch over e_count of the layer's E experts, of max_rows rows in all, and whether the
    down-projection runs in narrow units."""
    cfg, out = M.MoeCfg.make(T, d, f, E, k, "bf16"), (ctypes.c_int * 3)()
    lib().tile_rows(ctypes.addressof(cfg), gather, N_CU, E if e_count is None else e_count, T * k if max_rows is None else max_rows, out)
    return out[0], out[1], bool(out[2])
