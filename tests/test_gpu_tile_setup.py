"""The ILU(0) setup on the tiles: the factors and the numbers of dependency
levels against the level-by-level form (FAMS_ILU_RANGE=0), bit for bit, also
after new values on the kept schedule."""
import numpy as np
import pytest

from tests.test_gpu_tiles import _system

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", ["boxes", "flat", "2d", "dense", "wells", "shuffled",
                                  "shuffled-wells"])
def test_factors_and_levels(name, monkeypatch):
    from paper_1705_05784_amd import fams
    s, (wb, pr, vx, _) = _system(name)
    print(f"[tile setup] {name} n {s.n}", flush=True)

    def solver(val):
        return fams.Solver(s.row_ptr, s.col, val, s.n_matrix, wb, pr, vx, variant=0,
                           n_wells=s.n_wells)
    new = s.val * 1.25
    monkeypatch.delenv("FAMS_ILU_RANGE", raising=False)
    a = solver(s.val)
    lu = [a.ilu()]
    a.update_values(new, 10.0)
    lu.append(a.ilu())
    info = a.setup_info()
    monkeypatch.setenv("FAMS_ILU_RANGE", "0")
    for val, f in zip((s.val, new), lu):
        b = solver(val)
        assert np.array_equal(f, b.ilu())
        for k in ("ilu_levels_lower", "ilu_levels_upper"):
            assert info[k] == b.setup_info()[k] > 0, k
