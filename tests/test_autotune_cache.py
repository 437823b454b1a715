"""The autotuner's cache file without a GPU: entries of the present kernels are used without any device call, those
of earlier kernels, whose keys had no generation, are not.
"""
import ctypes

import pytest


def _call(P, path):
    from test_abi import _job
    best = P.Opts()
    arr = (type(_job()) * 1)(_job())
    st = P.lib().rs_autotune_batched(arr, 1, ctypes.c_void_p(0x4000), 1 << 20, None, str(path).encode(), ctypes.byref(best))
    return st, best


def test_entries_of_earlier_kernels_are_not_used(tmp_path):
    import torch
    if torch.cuda.is_available():
        pytest.skip("host check: the addresses are not real")
    import paper_0905_2453_amd as P
    key = "lens2^3|rays2^12|map2^8"
    cache = tmp_path / "tune.txt"
    cache.write_text(f"unknown|k2|{key} 2 4 512 32\n")
    st, best = _call(P, cache)
    assert st == 0 and (best.block_cols, best.block_rows, best.lens_tile, best.map_window) == (2, 4, 512, 32)
    cache.write_text(f"unknown|{key} 2 4 512 32\n")
    st, best = _call(P, cache)
    assert st == -3 and (best.block_cols, best.lens_tile) == (0, 0)      # it goes on to time candidates: no device
    assert cache.read_text().count("\n") == 1
