"""Which kernel the dense form runs follows the choice that callers make and see
(no GPU): the threshold scan is the last listed shape and the default, and every
compiled shape, the first among them, can be selected in its place.
"""
import ctypes
import os

import pytest

import paper_2008_05612_amd as hp


@pytest.fixture(scope="module")
def scans():
    if not os.path.exists(hp.library_path()):
        from paper_2008_05612_amd import build
        build.build()
    fn = getattr(hp.library(), "_ZN5hpmap10gemm_scansEi")   # the library's own rule, by depth / 32
    fn.restype, fn.argtypes = ctypes.c_bool, [ctypes.c_int]
    return fn


@pytest.mark.parametrize("K_pad", [32, 160, 192, 320, 384])
def test_every_listed_shape_can_be_selected(scans, K_pad):
    shapes = hp.hp_gemm_shapes(K_pad)
    keep = hp.hp_gemm_selected(K_pad)
    assert keep == len(shapes) - 1 and scans(K_pad // 32)
    assert [s[2] == 3 for s in shapes] == [False] * keep + [True]
    try:
        for i in range(len(shapes)):
            hp.hp_gemm_select(K_pad, i)
            assert hp.hp_gemm_selected(K_pad) == i
            assert scans(K_pad // 32) == (i == keep)
    finally:
        hp.hp_gemm_select(K_pad, keep)
    assert hp.hp_gemm_selected(K_pad) == keep and scans(K_pad // 32)
    for bad in (-1, len(shapes)):
        with pytest.raises(hp.HPError):
            hp.hp_gemm_select(K_pad, bad)
