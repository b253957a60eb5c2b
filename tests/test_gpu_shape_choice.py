"""Autotuning and the choices that it leaves: what it recorded is what a later
process reads, a handle that the scan does not cover leaves the scan to the
others, and a tuned blocked form still hands few sequences to the scan."""
import ctypes

import pytest

import paper_2008_05612_amd as hp
from tests.conftest import gpu_available

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not gpu_available():
        pytest.skip("no GPU")


def test_autotune_records_its_choice(tmp_path, monkeypatch):
    import torch
    s = hp.Structures(5, 5, 1)
    shapes = hp.hp_gemm_shapes(s.K_pad)
    keep = hp.hp_gemm_selected(s.K_pad)
    cache = tmp_path / "tuned"
    cache.write_text("gfx950 %d 1 1 1\ngfx950 32 4 4 0\n" % s.K_pad)   # its depth, and another
    monkeypatch.setenv("HP_TUNE_CACHE", str(cache))
    try:
        print("autotune", s.K_pad, flush=True)
        best, ms = hp.hp_autotune(s, s.workspace(), 0, 1 << 16, repeats=1)
        torch.cuda.synchronize()
    finally:
        hp.hp_gemm_select(s.K_pad, keep)
    compiled = ms[:-1].index(min(ms[:-1]))
    assert best == (len(shapes) - 1 if ms[-1] < ms[compiled] else compiled)
    assert cache.read_text().splitlines() == [
        "gfx950 32 4 4 0",
        "gfx950 %d %d %d %d %d" % ((s.K_pad,) + shapes[compiled] + (best == len(shapes) - 1,))]


class _Variant(ctypes.Structure):
    _fields_ = [("KB", ctypes.c_int), ("T", ctypes.c_int), ("NW", ctypes.c_int),
                ("mode", ctypes.c_int)]


def test_autotune_of_an_uncovered_table_leaves_the_scan_on():
    import torch
    scans = getattr(hp.library(), "_ZN5hpmap10gemm_scansEi")
    scans.restype = ctypes.c_bool
    variant = getattr(hp.library(), "_ZN5hpmap21gemm_selected_variantEi")
    variant.restype = ctypes.POINTER(_Variant)
    s = hp.Structures(5, 5, 1, table=(0, -32, -32, -72))     # B > 15
    assert s.K_pad == hp.Structures(3, 3, 3).K_pad           # which the scan covers
    shapes = hp.hp_gemm_shapes(s.K_pad)
    keep = hp.hp_gemm_selected(s.K_pad)
    assert keep == len(shapes) - 1
    print("autotune", s.K_pad, flush=True)
    best, ms = hp.hp_autotune(s, s.workspace(), 0, 1 << 16, repeats=1)
    torch.cuda.synchronize()
    assert ms[-1] == -1 and ms[best] == min(ms[:-1])
    hp.hp_gemm_select(s.K_pad, 0)
    hp.hp_gemm_select(s.K_pad, keep)      # as a caller that keeps and restores the choice
    v = variant(s.K_pad // 32).contents
    assert (v.T, v.NW, v.mode) == shapes[best]
    assert hp.hp_gemm_selected(s.K_pad) == keep and scans(s.K_pad // 32)


def test_tuned_blocks_leave_few_sequences_to_the_scan():
    import torch
    chosen = getattr(hp.library(), "_ZN5hpmap20blocked_shape_chosenEv")
    chosen.restype = ctypes.c_bool
    keep = hp.hp_blocked_selected()
    assert keep == (4, -1) and not chosen()
    try:
        hp.hp_blocked_select(4, 3)
        assert chosen()
        s = hp.Structures(5, 5, 1)
        print("autotune blocked", s.K_pad, flush=True)
        (nw, mode), _ = hp.hp_autotune_blocked(s, s.workspace(), 0, 1 << 18, repeats=1)
        torch.cuda.synchronize()
        assert mode >= 0 and hp.hp_blocked_selected() == (nw, mode)
        assert not chosen()
    finally:
        hp.hp_blocked_select(*keep)
    assert not chosen()
