"""The forms that lock-step sweeps choose from: pieces of a row twice as wide
(FAMS_SWEEP_WIDE, bytes of a vector from which they are taken) give the same
bits, as every row's arithmetic is the same; and where the level chunks are the
faster form (no grid behind the matrix rows, wide rows) they are taken, each
column within the bounds of the lock-step tests of its own single solve."""
import dataclasses

import numpy as np
import pytest
import scipy.sparse as sp

from tests.test_gpu_tiles import _system
from workloads import make_config

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

ONCE = dict(outer="richardson", rtol=0.0, max_iter=2)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("name", ["boxes", "flat", "2d", "dense", "wells", "shuffled-wells"])
def test_wide_pieces(name, precision, monkeypatch):
    from paper_1705_05784_amd import fams
    s, (wb, pr, vx, _) = _system(name)
    Q = torch.from_numpy(np.random.default_rng(5).standard_normal((32, s.n)))
    out = []
    for wide in (None, "0"):
        if wide is None:
            monkeypatch.delenv("FAMS_SWEEP_WIDE", raising=False)
        else:
            monkeypatch.setenv("FAMS_SWEEP_WIDE", wide)
        g = fams.Solver(s.row_ptr, s.col, s.val, s.n_matrix, wb, pr, vx, variant=0,
                        precision=precision, n_wells=s.n_wells)
        for k in (8, 16, 32):
            print(f"[block forms] {name} precision {precision} K {k} wide {wide}", flush=True)
            for _ in range(2):
                out.append(g.solve(Q[:k].contiguous(), **ONCE)[0].cpu().numpy())
        g.close()
    for a, b in zip(out[:6], out[6:]):
        assert np.array_equal(a, b)


def test_level_chunks_without_a_grid():
    """0.62M rows with one coupling out of place, FP64: 8 right-hand sides take
    the tiles, 32 the level chunks."""
    from paper_1705_05784_amd import fams
    s = make_config(2)
    wb, pr, vx, _ = fams.full_grid(s, (10, 10, 10), 8, 8)
    i = 5 * s.nx * s.ny + 5 * s.nx + 50
    j = 20 * s.nx * s.ny + 30 * s.nx + 10
    t = 1e-3
    A = (s.csr() + sp.coo_matrix(([-t, -t, t, t], ([i, j, i, j], [j, i, i, j])),
                                 shape=(s.n, s.n)).tocsr()).tocsr()
    A.sort_indices()
    s = dataclasses.replace(s, row_ptr=A.indptr.astype(np.int64),
                            col=A.indices.astype(np.int32), val=A.data.astype(np.float64))
    g = fams.Solver(s.row_ptr, s.col, s.val, s.n_matrix, wb, pr, vx, variant=0)
    Q = torch.from_numpy(np.random.default_rng(5).standard_normal((32, s.n))).cuda()
    one = [g.solve(Q[r], **ONCE)[0] for r in range(4)]
    for k in (8, 32, 8):
        print(f"[block forms] one coupling out of place, K {k}", flush=True)
        g.solve(Q[:k].contiguous(), **ONCE)   # builds what this width keeps
        g.profiling(True)
        P = g.solve(Q[:k].contiguous(), **ONCE)[0]
        assert ("bilu_arm" in g.kernel_stats()) == (k == 32)   # armed anew by each chunk sweep
        g.profiling(False)
        for r in range(4):
            d = float((P[r] - one[r]).abs().max())
            assert d <= 1e-10 * float(one[r].abs().max()), (k, r, d)
    g.close()
