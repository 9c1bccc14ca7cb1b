"""Tile schedules of rows whose order is found by their dependency levels, where
a key of tile and level would not hold it: more levels than a key has bits for
(a chain of 40,000 cells in tiles of one row).  The oracle is the level-by-level
form of the sweeps and of the factorisation (FAMS_ILU_RANGE=0), bit for bit."""
import numpy as np
import pytest

from tests._cases import homogeneous

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
        g.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b)
    assert out[0][2] == [s.n, s.n]
