"""Tile schedules of rows whose order is found by their dependency levels, where
a key of tile and level would not hold it: more levels than a key has bits for
(a chain of 40,000 cells in tiles of one row), and patterns that are not
symmetric, where the levels of the lower triangle are no order for the upper
one.  The oracle is the level-by-level form of the sweeps and of the
factorisation (FAMS_ILU_RANGE=0), bit for bit; for several right-hand sides the
single solves, within the bounds of the lock-step tests."""
import dataclasses

import numpy as np
import pytest
import scipy.sparse as sp

from tests._cases import homogeneous, small_case
from tests.test_gpu_tiles import _shuffled

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1])
def test_more_levels_than_key_bits(precision, monkeypatch):
    from paper_1705_05784_amd import fams
    s = homogeneous(40000, 1, 1, neumann=False)
    wb, pr, vx, _ = fams.full_grid(s, (100, 1, 1), 4, 1)
    r = torch.from_numpy(np.random.default_rng(5).standard_normal(s.n))
    out = []
    for rows in ("1", "0"):
        print(f"[tile orders] chain of {s.n}, precision {precision}, rows a tile {rows}", flush=True)
        monkeypatch.setenv("FAMS_ILU_RANGE", rows)
        g = fams.Solver(s.row_ptr, s.col, s.val, s.n_matrix, wb, pr, vx, precision=precision)
        info = g.setup_info()
        out.append((g.ilu(), g.apply_stage(r).cpu().numpy(),
                    [info["ilu_levels_lower"], info["ilu_levels_upper"]]))
        assert ("ilu_sum" in _kernels(g, r)) == (rows != "0")   # tiled sweeps
        g.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b)
    assert out[0][2] == [s.n, s.n]


def _one_sided(s, wb, lo, seed):
    """s with couplings stored on one side only (each row's diagonal grows by as
    much), above the diagonal and some below, between unknowns i, j >= lo with a
    common neighbour, all three of one medium and one wirebasket class: inside
    a local block, whose cells the symmetric couplings connect."""
    A = s.csr()
    rng = np.random.default_rng(seed)
    cls = np.asarray(wb) + 10 * (np.arange(s.n) >= s.n_matrix)
    r, c = A.nonzero()
    k = (r != c) & (r >= lo) & (c >= lo) & (cls[r] == cls[c])
    G = sp.csr_matrix((np.ones(k.sum()), (r[k], c[k])), shape=A.shape)
    i, j = sp.triu(G @ G, 1).nonzero()
    new = (np.asarray(A[i, j]).ravel() == 0) & (rng.random(len(i)) < 0.1)
    i, j = i[new], j[new]
    down = rng.random(len(i)) < 0.2
    i, j = np.where(down, j, i), np.where(down, i, j)
    t = np.abs(A.diagonal())[i] * 0.1 * rng.random(len(i))
    B = sp.coo_matrix((np.concatenate([-t, t]), (np.concatenate([i, i]), np.concatenate([j, i]))),
                      shape=A.shape)
    A = (A + B.tocsr()).tocsr()
    A.sort_indices()
    assert len(i) > 10 and ((A != 0) != (A != 0).T).nnz > 0
    return dataclasses.replace(s, row_ptr=A.indptr.astype(np.int64),
                               col=A.indices.astype(np.int32), val=A.data.astype(np.float64))


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("name", ["fractures", "matrix", "shuffled"])
@pytest.mark.parametrize("rows", [None, "64"])
def test_one_sided_couplings(rows, name, precision, monkeypatch):
    from paper_1705_05784_amd import fams
    s, spec = small_case("3d")
    grid = fams.full_grid(s, spec["coarse"], spec["d_min"], spec["r_z"])
    if name == "shuffled":
        s, grid = _shuffled(s, grid)
    wb, pr, vx, _ = grid
    s = _one_sided(s, wb, s.n_matrix if name == "fractures" else 0, 7)
    Q = torch.from_numpy(np.random.default_rng(5).standard_normal((4, s.n)))
    out = []
    for r in (rows, "0"):
        print(f"[tile orders] one-sided {name} precision {precision} rows a tile {r}", flush=True)
        if r is None:
            monkeypatch.delenv("FAMS_ILU_RANGE", raising=False)
        else:
            monkeypatch.setenv("FAMS_ILU_RANGE", r)
        g = fams.Solver(s.row_ptr, s.col, s.val, s.n_matrix, wb, pr, vx, precision=precision,
                        nonsymmetric=True)
        info = g.setup_info()
        one = [g.solve(q, outer="richardson", rtol=0.0, max_iter=1)[0].cpu().numpy() for q in Q]
        out.append((g.ilu(), g.apply_stage(Q[0]).cpu().numpy(), np.stack(one),
                    [info["ilu_levels_lower"], info["ilu_levels_upper"]]))
        if r != "0":
            assert "ilu_sum" in _kernels(g, Q[0])   # a launch of the tiled sweeps alone
        P = g.solve(Q, outer="richardson", rtol=0.0, max_iter=1)[0].cpu().numpy()
        tol = 1e-3 if precision else 1e-10
        for k in range(4):
            assert np.abs(P[k] - one[k]).max() <= tol * np.abs(one[k]).max()
        g.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b)


def _kernels(g, r):
    g.profiling(True)
    g.apply_stage(r)
    k = g.kernel_stats()
    g.profiling(False)
    return k


def test_waits_for_a_long_chain_are_not_long_waits(monkeypatch):
    """Every workgroup in flight waits for all the tiles before it: in a chain in
    tiles of eight rows for hundreds of hand-overs, over 1 ms, with nothing
    wrong.  long_waits counts workgroups that are not running (from 8 ms on)."""
    from paper_1705_05784_amd import fams
    s = homogeneous(40000, 1, 1, neumann=False)
    wb, pr, vx, _ = fams.full_grid(s, (100, 1, 1), 4, 1)
    monkeypatch.setenv("FAMS_ILU_RANGE", "8")
    g = fams.Solver(s.row_ptr, s.col, s.val, s.n_matrix, wb, pr, vx)
    Q = torch.from_numpy(np.random.default_rng(5).standard_normal((8, s.n)))
    for k in (1, 2, 8):
        g.solve(Q[:k].contiguous() if k > 1 else Q[0], outer="richardson", rtol=0.0, max_iter=2)
        print(f"[tile orders] {k} right-hand sides, long waits {g.setup_info()['long_waits']}",
              flush=True)
    assert g.setup_info()["long_waits"] == 0
    g.close()
