"""The tiled sweeps' divisions by the diagonal at the ends of the numbers' range:
quotients that overflow, small inputs (down to where the residual of an FP64
quotient is exact, and around the smallest normal number of either precision),
diagonals whose reciprocal lies below the smallest normal number.  The oracle is the level-by-level form
(FAMS_ILU_RANGE=0), which divides: the same bits, infinities included; in
lock-step the single step's infinities."""
import dataclasses

import numpy as np
import pytest

from tests._cases import small_case

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

MAX = {0: float(np.finfo(np.float64).max), 1: float(np.finfo(np.float32).max)}


def _weak_cell(s, c, f):
    """s with all couplings of cell c times f (row sums kept)."""
    A = s.csr().tolil()
    for j in list(A.rows[c]):
        if j != c:
            t = -A[c, j]
            A[c, j] = A[j, c] = -f * t
            A[c, c] -= (1 - f) * t
            A[j, j] -= (1 - f) * t
    return _with(s, A.tocsr())


def _with(s, A):
    A.sort_indices()
    return dataclasses.replace(s, row_ptr=A.indptr.astype(np.int64),
                               col=A.indices.astype(np.int32), val=A.data.astype(np.float64))


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("kind", ["overflow", "tiny", "tiniest", "large diagonal"])
def test_division_at_the_ends(kind, precision, monkeypatch):
    from paper_1705_05784_amd import fams
    s, spec = small_case("3d")
    wb, pr, vx, _ = fams.full_grid(s, spec["coarse"], spec["d_min"], spec["r_z"])
    r = np.random.default_rng(5).standard_normal(s.n)
    if kind == "overflow":
        c = s.n_matrix // 2 + s.nx // 2
        s = _weak_cell(s, c, 1e-7)
        r = np.zeros(s.n)
        r[c] = 4.0 * s.csr()[c, c] * MAX[precision]
    elif kind == "tiny":
        r *= 2.0 ** (-135 if precision else -900)
    elif kind == "tiniest":
        r *= 2.0 ** (-145 if precision else -1020)
    else:   # diagonals up to the largest power of two; small inputs, so that nothing overflows
        e = (126 if precision else 1022) - int(np.ceil(np.log2(s.csr().diagonal().max())))
        s = _with(s, s.csr() * 2.0 ** e)
        r *= 2.0 ** (e - 20)
    r = torch.from_numpy(r)
    z = []
    for rows in (None, "0"):
        print(f"[sweep range] {kind} precision {precision} rows {rows}", flush=True)
        if rows is None:
            monkeypatch.delenv("FAMS_ILU_RANGE", raising=False)
        else:
            monkeypatch.setenv("FAMS_ILU_RANGE", rows)
        g = fams.Solver(s.row_ptr, s.col, s.val, s.n_matrix, wb, pr, vx, precision=precision)
        z.append(g.apply_stage(r).cpu().numpy())
        if rows is None and precision and kind == "overflow":   # q . q is finite in FP64
            P = g.solve(torch.stack([r, r]), outer="richardson", rtol=0.0, max_iter=1)[0]
            for p in P.cpu().numpy():
                assert np.array_equal(np.isposinf(p), np.isposinf(z[0]))
                assert np.array_equal(np.isfinite(p), np.isfinite(z[0]))
        g.close()
    assert np.array_equal(z[0], z[1], equal_nan=True)
    if kind == "overflow":
        assert np.isposinf(z[1]).sum() > 1 and np.isfinite(z[1]).any()
    else:
        assert np.isfinite(z[1]).all()
