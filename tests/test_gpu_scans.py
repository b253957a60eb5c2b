"""The threshold scans against the oracle, and against the popcount form where
the oracle would take too long: ranges at the edges of tiles, blocks, chunks
and launch shapes, pure pair energies and two-letter tables, all outputs.
Every output is a whole number, so each comparison is exact.  Besides, the
network passes on maps that fill their edge lists and on unaligned buffers.
"""
import numpy as np
import pytest

import oracle
import paper_2008_05612_amd as hp
from tests.conftest import gpu_available

pytestmark = pytest.mark.gpu
HP1996 = oracle.HP1996_X10
T2 = (0, -1, -1, -3)
NONE = 0xFFFF
_cache = {}


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not gpu_available():
        pytest.skip("no GPU")


def _get(dims, table):
    key = (dims, table)
    if key not in _cache:
        s = hp.Structures(*dims, table=table)
        _cache[key] = (s, s.workspace())
    return _cache[key]


def _run(dims, table, form, lo, n, threshold, shape=None):
    """[out, emin, gap, designability, nondesign] of [lo, lo + n)."""
    import torch
    s, ws = _get(dims, table)
    o = torch.full((n,), -7, dtype=torch.int16, device="cuda")
    e = torch.full((n,), 99, dtype=torch.int32, device="cuda")
    g = torch.zeros(n, dtype=torch.uint8, device="cuda")
    d = torch.zeros(s.n_class, dtype=torch.int64, device="cuda")
    nd = torch.zeros(1, dtype=torch.int64, device="cuda")
    print("scan", dims, table, form, lo, n, threshold, shape, flush=True)
    if shape:
        hp.hp_blocked_select(*shape)
    try:
        hp.hp_enumerate_gap(s, ws, form, lo, lo + n, threshold, o, e, g, d, nd)
        torch.cuda.synchronize()
    finally:
        if shape:
            hp.hp_blocked_select(4, -1)
    return [t.cpu().numpy() for t in (o, e, g, d, nd)]


def _same(a, b):
    for x, y in zip(a, b):
        assert np.array_equal(x, y)


# Dense scan: one sequence to its largest shapes.  The lines lie at 32 and 64
# columns, at 8192 and 16384 sequences, and where the blocks take over.
@pytest.mark.parametrize("n", [1, 31, 32, 33, 63, 65, 1000, 8191, 8193, 16384, 16385, 79999])
@pytest.mark.parametrize("table", [None, HP1996, T2])
def test_dense_scan_sizes(table, n):
    dims = (5, 4, 1)
    lo = 777
    want = _run(dims, table, hp.FORM_POPCOUNT, lo, n, 2)
    _same(_run(dims, table, hp.FORM_BLOCKED_I8, lo, n, 2), want)
    _same(_run(dims, table, hp.FORM_GEMM_I8, lo, n, 2), want)
    w = min(n, 512)
    gs = oracle.ground_states_gap(oracle.structures(*dims), np.arange(lo, lo + w, dtype=np.uint64),
                                  2, table=table)
    assert np.array_equal(want[0][:w].view(np.uint16), gs.out)
    assert np.array_equal(want[1][:w], gs.emin)


# Blocks: few (their conformations split), a ragged pair, either side of the
# line of few-class boxes, and ranges holding chunks of 2^19 and 2^17 and loose
# blocks on both sides of them; 5x5 counts its classes in LDS, 2x3x4 does not.
@pytest.mark.parametrize("dims,lo,n", [
    ((5, 5, 1), 1023, 2), ((5, 5, 1), 1000, 90001), ((5, 5, 1), 5, 384 * 1024),
    ((5, 5, 1), 5, 385 * 1024), ((5, 5, 1), (1 << 19) - 70001, (1 << 21) + 300007),
    ((2, 3, 4), 3, 150001), ((2, 3, 4), (1 << 19) - 140007, (1 << 21) + 300011),
    ((2, 3, 4), 0, 1 << 21)])
@pytest.mark.parametrize("table", [None, HP1996])
def test_wide_scan_ranges(table, dims, lo, n):
    s, _ = _get(dims, table)
    lo = min(lo, (1 << s.N) - n)
    want = _run(dims, table, hp.FORM_POPCOUNT, lo, n, 3)
    _same(_run(dims, table, hp.FORM_BLOCKED_I8, lo, n, 3), want)           # by size
    _same(_run(dims, table, hp.FORM_BLOCKED_I8, lo, n, 3, (4, 3)), want)   # blocks of 1024
    w = min(n, 256)
    st = oracle.structures(*dims)
    for off in (0, n - w):
        gs = oracle.ground_states(st, lo + off, lo + off + w, table=table)
        assert np.array_equal(want[1][off:off + w], gs.emin)


def _network(s, phen, offset):
    """(labels, sizes, phi counts) with the map, the labels and the matrix
    `offset` elements off their buffers' starts."""
    import torch
    n = 1 << s.N
    view = torch.zeros(n + 16, dtype=torch.int16, device="cuda")[offset:offset + n]
    view.copy_(torch.from_numpy(phen.view(np.int16)))
    lab = torch.zeros(n + 16, dtype=torch.int32, device="cuda")[offset:offset + n]
    size = torch.zeros(n, dtype=torch.int32, device="cuda")
    ncomp = torch.zeros(s.n_class, dtype=torch.int32, device="cuda")
    largest = torch.zeros(s.n_class, dtype=torch.int32, device="cuda")
    print("network", s.N, offset, flush=True)
    hp.hp_components(s, view, lab, size, ncomp, largest)
    m = s.n_class * (s.n_class + 1)
    counts = torch.zeros(m + 16, dtype=torch.int64, device="cuda")[offset:offset + m]
    counts = counts.view(s.n_class, s.n_class + 1)
    hp.hp_phi_counts(s, view, counts)
    rp = torch.zeros(s.n_class + 1, dtype=torch.int64, device="cuda")
    nnz = hp.hp_phi_sparse(s, counts, rp)
    cols = torch.zeros(nnz, dtype=torch.int32, device="cuda")
    vals = torch.zeros(nnz, dtype=torch.int64, device="cuda")
    hp.hp_phi_sparse(s, counts, rp, cols, vals)
    torch.cuda.synchronize()
    return [t.cpu().numpy() for t in (lab, size, ncomp, largest, counts, rp, cols, vals)]


# One phenotype everywhere (every mutant an edge), along the low bits alone, and
# half of it; 8 genotypes is the smallest map of the vector path.
@pytest.mark.parametrize("dims", [(3, 1, 1), (2, 2, 1), (3, 3, 1), (3, 4, 1), (4, 4, 1)])
@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("kind", ["full", "vectors", "half"])
def test_network_dense_maps(dims, offset, kind):
    try:
        s = hp.Structures(*dims)
    except hp.HPError:
        pytest.skip("no such box")
    n = 1 << s.N
    g = np.arange(n)
    rng = np.random.default_rng(s.N)
    phen = np.zeros(n, dtype=np.uint16)
    if kind == "vectors":
        phen = (np.array([bin(x >> 3).count("1") for x in g]) % 2 % s.n_class).astype(np.uint16)
    elif kind == "half":
        phen[rng.random(n) < 0.5] = NONE
    lab, size, ncomp, largest, counts, rp, cols, vals = _network(s, phen, offset)
    want = oracle.components(s.N, phen)
    assert np.array_equal(lab.view(np.uint32), want)
    des = phen != NONE
    sizes = np.bincount(want[des], minlength=n)
    assert np.array_equal(size, sizes)
    roots = des & (want == g)
    assert np.array_equal(ncomp, np.bincount(phen[roots], minlength=s.n_class))
    assert largest[0] == (sizes[roots & (phen == 0)].max() if (roots & (phen == 0)).any() else 0)
    dense = oracle.phi_counts(s.N, phen, s.n_class)
    assert np.array_equal(counts.view(np.uint64), dense)
    rows, c = np.nonzero(dense)
    assert np.array_equal(cols.view(np.uint32), c)
    assert np.array_equal(vals.view(np.uint64), dense[rows, c])
    assert np.array_equal(rp, np.concatenate([[0], np.cumsum(np.count_nonzero(dense, axis=1))]))
