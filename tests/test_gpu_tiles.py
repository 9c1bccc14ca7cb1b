"""The tiled ILU(0) sweeps where their schedule has edges: boxes cut by the
grid's sides in every direction, lines shorter than a box, 2D grids, networks
with many intersections (eight dependency places a row, and the terms beyond
them), wells, and matrix cells in an order that is no grid (one phase of
consecutive rows).  The oracle is the level-by-level form of the same sweeps
(FAMS_ILU_RANGE=0): every row's terms are subtracted in the same order, so the
two-stage step has the same bits."""
import dataclasses

import numpy as np
import pytest

from tests._cases import small_case, wells_case
from workloads import make_config, make_small

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _shuffled(s, grid):
    """The system with its matrix cells in a random order."""
    wb, pr, vx, _ = grid
    perm = np.arange(s.n)
    perm[:s.n_matrix] = np.random.default_rng(3).permutation(s.n_matrix)
    inv = np.empty_like(perm)
    inv[perm] = np.arange(s.n)
    A = s.csr()[perm][:, perm].tocsr()
    A.sort_indices()
    s2 = dataclasses.replace(s, row_ptr=A.indptr.astype(np.int64), col=A.indices.astype(np.int32),
                             val=A.data.astype(np.float64))
    return s2, (np.asarray(wb)[perm], np.asarray(pr)[perm], inv[np.asarray(vx)], None)


def _system(name):
    from paper_1705_05784_amd import fams
    if name.startswith("shuffled"):
        s, spec = wells_case("3d") if name.endswith("wells") else small_case("3d")
    elif name == "wells":
        s, spec = wells_case("cfg2s")
    elif name == "2d":
        s, spec = make_config(1, 7, dims=(130, 71, 1)), dict(coarse=(10, 10, 1), d_min=10, r_z=1)
    elif name == "boxes":   # two boxes along x, odd remainders along y and z
        s, spec = make_small("3d", nx=131, ny=19, nz=17, n_frac=8, len3d=(8, 30)), None
    elif name == "flat":    # fewer lines along z than a box holds
        s, spec = make_small("3d", nx=9, ny=70, nz=3, n_frac=4, h3d=(2, 3)), None
    else:                   # dense network: many intersections
        s, spec = make_small("3d", nx=24, ny=22, nz=12, n_frac=60, len3d=(8, 20)), None
    spec = spec or dict(coarse=(4, 4, 4), d_min=4, r_z=4)
    g = fams.full_grid(s, spec["coarse"], spec["d_min"], spec["r_z"])
    return _shuffled(s, g) if name.startswith("shuffled") else (s, g)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("name", ["boxes", "flat", "2d", "dense", "wells", "shuffled",
                                  "shuffled-wells"])
def test_tiled_sweeps(name, precision, monkeypatch):
    from paper_1705_05784_amd import fams
    s, (wb, pr, vx, _) = _system(name)
    print(f"[tiles] {name} precision {precision} n {s.n}", flush=True)

    def solver(**kw):
        return fams.Solver(s.row_ptr, s.col, s.val, s.n_matrix, wb, pr, vx, variant=0,
                           precision=precision, n_wells=s.n_wells, **kw)
    r = torch.from_numpy(np.random.default_rng(5).standard_normal(s.n))
    for smoother in (1, 2):   # 2: the second stage's own factors and schedule
        monkeypatch.delenv("FAMS_ILU_RANGE", raising=False)
        a = solver(smoother=smoother)
        za = [a.apply_stage(r).cpu().numpy() for _ in range(2)]   # the second re-uses the state
        monkeypatch.setenv("FAMS_ILU_RANGE", "0")
        zb = solver(smoother=smoother).apply_stage(r).cpu().numpy()
        assert np.isfinite(zb).all()
        assert np.array_equal(za[0], zb)
        assert np.array_equal(za[1], zb)
