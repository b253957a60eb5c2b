"""The threshold scans at the launch shapes and product depths that the other
boxes do not reach, against the popcount form (exact integers by another route)
and, over windows, the oracle: the split shapes on both sides of their lines, odd
numbers of conformation tiles, chains of 28 to 35 monomers, and two-letter
tables beyond the dense scan's bounds, which run the int8 shapes.
"""
import numpy as np
import pytest

import oracle
import paper_2008_05612_amd as hp
from tests.conftest import gpu_available
from tests.test_gpu_scans import _get, _run, _same

pytestmark = pytest.mark.gpu
HP1996 = oracle.HP1996_X10


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not gpu_available():
        pytest.skip("no GPU")


def _oracle_window(dims, table, lo, got, w):
    gs = oracle.ground_states_gap(oracle.structures(*dims), np.arange(lo, lo + w, dtype=np.uint64),
                                  2, table=table)
    assert np.array_equal(got[0][:w].view(np.uint16), gs.out)
    assert np.array_equal(got[1][:w], gs.emin)
    assert np.array_equal(got[2][:w], gs.gap)


# Conformations split over 8 or 16 waves (16 steps and more): 32 columns per
# workgroup up to 8192 sequences, 64 beyond, and four waves per SIMD up to 16384
# where the chain is short.  2x3x3 has 66 tiles, 5x5 34, 6x4 an odd 57, 6x6 1792;
# pure chains of 3, 5, 4 and 10 products.
@pytest.mark.parametrize("n", [1, 32, 33, 65, 8191, 8192, 8193, 16384, 16385, 20001])
@pytest.mark.parametrize("dims", [(2, 3, 3), (5, 5, 1), (6, 4, 1), (6, 6, 1)])
@pytest.mark.parametrize("table", [None, HP1996])
def test_split_scan_lines(table, dims, n):
    s, _ = _get(dims, table)
    lo = int(0.7 * (1 << s.N))
    want = _run(dims, table, hp.FORM_POPCOUNT, lo, n, 2)
    _same(_run(dims, table, hp.FORM_GEMM_I8, lo, n, 2), want)
    if hp.hp_canonical_block_count(s):
        _same(_run(dims, table, hp.FORM_BLOCKED_I8, lo, n, 2), want)
    _oracle_window(dims, table, lo, want, min(n, 32))


# 28, 30, 32 .. 35 monomers: chains of 6 to 9 products (tables 4 and 5), and
# boxes of few conformations on both sides of 2^17 sequences, whose largest
# workgroups hold more than 64 KB of LDS.
DEEP = [(14, 2, 1), (7, 4, 1), (15, 2, 1), (10, 3, 1), (6, 5, 1), (16, 2, 1), (11, 3, 1), (8, 4, 1),
        (17, 2, 1), (7, 5, 1), (18, 2, 1)]


@pytest.mark.parametrize("n", [3001, (1 << 17) + 1, 300007])
@pytest.mark.parametrize("dims", DEEP)
@pytest.mark.parametrize("table", [None, HP1996])
def test_deep_chains(table, dims, n):
    s, _ = _get(dims, table)
    lo = int(0.7 * (1 << s.N))
    want = _run(dims, table, hp.FORM_POPCOUNT, lo, n, 2)
    _same(_run(dims, table, hp.FORM_GEMM_I8, lo, n, 2), want)
    if hp.hp_canonical_block_count(s):
        _same(_run(dims, table, hp.FORM_BLOCKED_I8, lo, n, 2, (4, 3)), want)   # blocks of 1024
    _oracle_window(dims, table, lo, want, 64)


# the largest blocks at those depths: a range that holds a chunk of 2^19, chunks
# of 2^17 and loose blocks on both sides
@pytest.mark.parametrize("dims", [(7, 4, 1), (10, 3, 1), (11, 3, 1), (17, 2, 1)])
def test_deep_wide_blocks(dims):
    s, _ = _get(dims, None)
    lo = ((int(0.7 * (1 << s.N)) >> 19) << 19) - 140007
    n = (1 << 21) + 300011
    want = _run(dims, None, hp.FORM_POPCOUNT, lo, n, 2)
    _same(_run(dims, None, hp.FORM_BLOCKED_I8, lo, n, 2, (8, 3)), want)


# reversal-canonical wide blocks at those depths: the first blocks have the h low
# monomers all P (block 0) or all H with the high ones counting up
@pytest.mark.parametrize("dims", [(14, 2, 1), (15, 2, 1), (16, 2, 1), (17, 2, 1), (11, 3, 1)])
def test_deep_canonical_wide_blocks(dims):
    import torch
    s, ws = _get(dims, None)
    odd = s.N & 1
    h = (s.N - 10 - odd) // 2
    x = np.arange(1024, dtype=np.uint64)
    mid = (x & np.uint64(31)) | ((x >> np.uint64(5)) << np.uint64(5 + odd))
    seqs = [(np.uint64(a) << np.uint64(h + 10 + odd)) | (mid << np.uint64(h)) | np.uint64(b)
            for a, b in ((0, 0), (0, (1 << h) - 1), (1, (1 << h) - 1), (2, (1 << h) - 1))]
    seqs = np.concatenate(seqs)
    rev = np.zeros_like(seqs)
    for i in range(s.N):
        rev |= ((seqs >> np.uint64(i)) & np.uint64(1)) << np.uint64(s.N - 1 - i)
    out = torch.empty(1 << s.N, dtype=torch.int16, device="cuda")
    desig = torch.zeros(s.n_class, dtype=torch.int64, device="cuda")
    nond = torch.zeros(1, dtype=torch.int64, device="cuda")
    print("canonical wide", dims, flush=True)
    hp.hp_enumerate_symmetric_wide(s, ws, 0, 4, out, None, desig, nond)
    got = [out[torch.from_numpy(q.view(np.int64)).cuda()].cpu().numpy().view(np.uint16)
           for q in (seqs, rev)]
    gs = oracle.ground_states_gap(oracle.structures(*dims), seqs, 1)
    assert np.array_equal(got[0], gs.out) and np.array_equal(got[1], gs.out)
    # block 0 holds both of every pair of reversed sequences, the others one of two
    weight = np.repeat([1, 2, 2, 2], 1024)
    none = gs.out == 0xFFFF
    assert int(nond.item()) == int(weight[none].sum())
    assert np.array_equal(desig.cpu().numpy(),
                          np.bincount(gs.out[~none], weights=weight[~none],
                                      minlength=s.n_class).astype(np.int64))


# Tables that the dense scan does not cover (B > 15): F to 1470 at the all-H end
# of the range, so that the blocks' threshold needs its upper digit; the dense
# form runs every compiled int8 shape.
@pytest.mark.parametrize("dims,table", [((5, 5, 1), (0, -32, -32, -72)),
                                        ((2, 3, 3), (0, -32, -32, -64)),
                                        ((6, 2, 2), (0, -32, -32, -70))])
@pytest.mark.parametrize("n", [2049, 100001])
def test_tables_beyond_the_scan(dims, table, n):
    s, _ = _get(dims, table)
    assert hp.hp_canonical_block_count(s)
    lo = (1 << s.N) - n
    want = _run(dims, table, hp.FORM_POPCOUNT, lo, n, 2)
    assert want[1].min() < -742
    _same(_run(dims, table, hp.FORM_BLOCKED_I8, lo, n, 2), want)
    _same(_run(dims, table, hp.FORM_BLOCKED_I8, lo, n, 2, (4, 2)), want)   # blocks of 256
    keep = hp.hp_gemm_selected(s.K_pad)
    try:
        for i in range(len(hp.hp_gemm_shapes(s.K_pad))):
            hp.hp_gemm_select(s.K_pad, i)
            _same(_run(dims, table, hp.FORM_GEMM_I8, lo, n, 2), want)
    finally:
        hp.hp_gemm_select(s.K_pad, keep)
    _oracle_window(dims, table, lo, want, 64)
