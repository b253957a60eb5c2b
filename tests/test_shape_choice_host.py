"""Which kernel the dense form runs follows the choice that callers make and see
(no GPU): the threshold scan is the last listed shape and the default, and every
compiled shape, the first among them, can be selected in its place.
"""
import ctypes
import os
import subprocess
import sys

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


_READ_BACK = """
import ctypes, paper_2008_05612_amd as hp
fn = getattr(hp.library(), "_ZN5hpmap10gemm_scansEi")
fn.restype = ctypes.c_bool
print(hp.hp_gemm_selected(160), fn(5), hp.hp_gemm_selected(192), fn(6))
"""


# A record of hp_autotune says whether its shape was faster than the scan; one
# without that field was timed without the scan.  A line of another kind is passed
# over.
@pytest.mark.parametrize("field,scan", [(" 0", False), (" 1", True), ("", True)])
def test_recorded_choice_is_read_back(tmp_path, field, scan):
    shapes = hp.hp_gemm_shapes(160)
    cache = tmp_path / "tuned"
    cache.write_text("# shapes\ngfx950 160 %d %d %d%s\n" % (shapes[2] + (field,)))
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    out = subprocess.run([sys.executable, "-c", _READ_BACK], capture_output=True, text=True,
                         cwd=root, env=dict(os.environ, HP_TUNE_CACHE=str(cache)))
    assert out.returncode == 0, out.stderr
    other = len(hp.hp_gemm_shapes(192)) - 1
    assert out.stdout.split() == [str(len(shapes) - 1 if scan else 2), str(scan), str(other), "True"]
