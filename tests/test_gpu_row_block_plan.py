"""The plan of the row blocks (general patterns), which the device makes at
every assembly.

Its cost: the same matrix is assembled as it is (rows of at most six
dependencies: row blocks) and with one row made wider than the row blocks take
(level sweeps); levels, factorization and packing are the same work, so the
plan has to cost no more than the level schedule.  Shortest of several
assemblies in turn, a fifth allowed for noise.

Its result, through the sweeps, where the lists of outside rows are longest
and most shared: every dependency in another block and another row (1 536
outside rows a block, the hash table three quarters full), one row read by all
of a block, blocks of a single row and of none beside full ones, numbers in
random and in red-black order.  Tolerance: diagonally dominant blocks, so the
FP64 apply differs from the oracle by a few ulps a row, far below 1e-12."""
import time

import numpy as np
import pytest

import oracle
import reservoir_inputs as ri

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1701_05913_amd as K  # noqa: E402
from tests.gpu_helpers import GpuSystem, make_solver, pc_apply, relerr  # noqa: E402


def _renumbered(s, new):
    """Row i of s as row new[i]."""
    bs = s.get("bs", 1)
    row = np.repeat(np.arange(new.size), np.diff(s["rowptr"]))
    r, c = new[row], new[s["col"]]
    order = np.lexsort((c, r))
    rowptr = np.zeros(new.size + 1, dtype=np.int32)
    rowptr[1:] = np.cumsum(np.bincount(r, minlength=new.size))
    val = np.asarray(s["val"]).reshape(-1, bs, bs)[order]
    return dict(rowptr=rowptr, col=c[order].astype(np.int32), val=val.reshape(-1), bs=bs)


def _with_wide_row(s):
    """Zero blocks added to the last row until it has eight lower neighbours."""
    bs, nb = s["bs"], s["rowptr"].size - 1
    p = int(s["rowptr"][nb - 1])
    have = s["col"][p:]
    low = have[have < nb - 1]
    more = np.setdiff1d(np.arange(0, nb - 1, max(1, nb // 16)), low)[:8 - low.size]
    col = np.concatenate([have, more])
    val = np.concatenate([s["val"][p * bs * bs:], np.zeros(more.size * bs * bs)]).reshape(-1, bs, bs)
    order = np.argsort(col)
    rowptr = s["rowptr"].copy()
    rowptr[nb] += more.size
    return dict(rowptr=rowptr, col=np.concatenate([s["col"][:p], col[order]]).astype(np.int32),
                val=np.concatenate([s["val"][:p * bs * bs], val[order].reshape(-1)]), bs=bs)


@pytest.mark.parametrize("order", ["redblack", "random"])
def test_row_blocks_cost_no_more_than_levels(order):
    nx, ny, nz = 48, 44, 40
    s = ri.blackoil_system(nx, ny, nz, seed=3)
    c = np.arange(nx * ny * nz)
    key = (c % nx + c // nx % ny + c // (nx * ny)) % 2 if order == "redblack" else \
        np.random.default_rng(5).permutation(c.size)
    new = np.empty_like(c)
    new[np.argsort(key, kind="stable")] = c
    s = _renumbered(dict(s, bs=3), new)
    systems = [GpuSystem(q) for q in (s, _with_wide_row(s))]
    solvers = [make_solver(g, K.KRY_GMRES, K.KRY_PC_BILU0) for g in systems]
    best = []
    try:
        for S, g in zip(solvers, systems):
            K.SolverSetMat(S, g.A)
            K.SolverAssemble(S)
        times = [[], []]
        for _ in range(7):
            for t, S in zip(times, solvers):
                torch.cuda.synchronize()
                t0 = time.perf_counter()
                K.SolverAssemble(S)
                torch.cuda.synchronize()
                t.append(time.perf_counter() - t0)
        best = [min(t) for t in times]
    finally:
        for S, g in zip(solvers, systems):
            K.SolverDestroy(S)
            g.close()
    print(f"{order}: row blocks {best[0] * 1e3:.2f} ms, levels {best[1] * 1e3:.2f} ms")
    assert best[0] <= 1.2 * best[1]


def _system(nb, entries, bs, seed):
    """Diagonally dominant matrix with the given off-diagonal entries."""
    rng = np.random.default_rng(seed)
    entries = np.unique(np.asarray(entries).reshape(-1, 2), axis=0)
    row = np.concatenate([entries[:, 0], np.arange(nb)])
    col = np.concatenate([entries[:, 1], np.arange(nb)])
    order = np.lexsort((col, row))
    row, col = row[order], col[order]
    rowptr = np.zeros(nb + 1, dtype=np.int32)
    rowptr[1:] = np.cumsum(np.bincount(row, minlength=nb))
    val = rng.uniform(-1.0, 1.0, (col.size, bs, bs)) * (0.5 / (12 * bs))
    val[col == row] += np.diag(1.0 + rng.random(bs))
    return dict(rowptr=rowptr, col=col.astype(np.int32), val=val.reshape(-1), bs=bs)


def _both(pairs):
    pairs = np.asarray(pairs).reshape(-1, 2)
    return np.concatenate([pairs, pairs[:, ::-1]])


def _far(nb):
    # row i reads one row of each of the six blocks before its own, every row
    # of a block others
    return _both([(i, i - i % 256 - 256 * q + (i + 37 * q) % 256)
                  for i in range(nb) for q in range(1, 7) if i >= 256 * (q + 1)])


def _shared(nb):
    # all rows of a block read the same six rows of the block before, and the
    # same three rows of the next one
    low = [(i, i - i % 256 - 1 - 40 * q) for i in range(256, nb) for q in range(6)]
    return low + [(i, k) for i in range(nb) for k in (i - i % 256 + 256 + 9 * q for q in range(3)) if k < nb]


def _reordered(nb, key):
    # a 7-point pattern (13 rows a line, 11 lines a layer) in the order of key
    new = np.empty(nb, dtype=np.int64)
    new[np.argsort(key, kind="stable")] = np.arange(nb)
    pairs = []
    for d, edge in ((1, 13), (13, 143), (143, nb + 1)):
        i = np.arange(d, nb)
        i = i[(i % edge) >= d]
        pairs.append(np.stack([new[i], new[i - d]], 1))
    pairs = np.concatenate(pairs)
    return _both(pairs)


PATTERNS = {
    "far_2304": (2304, _far(2304)),
    "far_2305": (2305, _far(2305)),
    "shared_1024": (1024, _shared(1024)),
    "shared_1537": (1537, _shared(1537)),
    "none_513": (513, np.zeros((0, 2), dtype=int)),
    "redblack_2574": (2574, _reordered(2574, (np.arange(2574) % 13 + np.arange(2574) // 13 % 11 + np.arange(2574) // 143) % 2)),
    "random_2574": (2574, _reordered(2574, np.random.default_rng(8).permutation(2574))),
}


@pytest.mark.parametrize("bs", [1, 3])
@pytest.mark.parametrize("name", list(PATTERNS))
def test_outside_rows(name, bs):
    nb, pairs = PATTERNS[name]
    s = _system(nb, pairs, bs, seed=nb)
    A = oracle.Matrix.from_system(s)
    v = np.random.default_rng(4).standard_normal(A.n)
    ref = oracle.PC(A, "bilu0").apply(v)
    g = GpuSystem(s)
    try:
        z1, z2 = pc_apply(g, K.KRY_PC_ILU0, v, layout=K.KRY_SWEEP_LEVELS, repeat=2)
    finally:
        g.close()
    assert relerr(z1, ref) <= 1e-12
    assert np.array_equal(z1, z2)
