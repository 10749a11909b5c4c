"""The workspace a call needs is part of the interface: a caller may keep a buffer of the size that a
program was told before, so the sizes stay what they were."""
import ctypes

import pytest

from paper_2007_03800_amd import _native

ONE, ODD = (8, 8, 16, 16, 8, 100000), [(9, 7, 13, 11, 6, 20011), (12, 12, 20, 20, 10, 5), (64, 2, 64, 3, 4, 300)]
SMALL = (4, 4, 6, 6, 3, 70)
# (problems, precision, call, K, bytes)
SIZES = [([], "fp64", 0, 0, 1032), ([], "fp32", 2, 7, 1088), ([ONE], "fp64", 0, 0, 3218632), ([ONE], "fp64", 2, 7, 3218632),
         ([ONE], "fp32", 1, 0, 3215560), ([ONE], "fp32", 3, 0, 3215560), ([(1, 1, 1, 1, 1, 0)], "fp64", 2, 7, 28424),
         (ODD, "fp64", 2, 7, 76086792), (ODD, "fp32", 0, 0, 76046856), ([SMALL] * 40, "fp64", 0, 0, 20450568),
         ([SMALL] * 40, "fp64", 2, 7, 20452616), ([SMALL] * 40, "fp32", 2, 7, 20432136)]


@pytest.mark.parametrize("shapes,prec,call,K,want", SIZES)
def test_workspace_bytes(shapes, prec, call, K, want):
    arr = (_native.Problem * max(1, len(shapes)))()
    at = ctypes.c_void_p(4096)  # sizes only: no buffer is touched
    for i, (m1, m2, n1, n2, s, N) in enumerate(shapes):
        arr[i] = _native.Problem(m1, m2, n1, n2, s, 0, N, at, at, at, at, at, at)
    o = _native.default_options()
    o.prec = {"fp64": _native.SDL_FP64, "fp32": _native.SDL_FP32}[prec]
    n = ctypes.c_size_t()
    assert _native.lib().sdl_workspace_bytes(arr, len(shapes), call, K, ctypes.byref(o), ctypes.byref(n)) == 0
    assert n.value == want
