"""The lock-step tiled ILU(0) sweeps on the systems of the single-vector ones,
at every group width: each column of one Richardson iteration from zero (one
application of the two-stage preconditioner) against its own single solve,
whose sweeps are bit-identical to the level-by-level form.  The sweeps subtract
every row's terms in the same order; the other kernels of the stage sum in
another order, which its well conditioned triangular and coarse solves keep
within some 1e3 rounding errors: 1e-10 in FP64 and 1e-3 with the FP32 stage."""
import numpy as np
import pytest

from tests.test_gpu_tiles import _system

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("name", ["boxes", "flat", "2d", "dense", "wells", "shuffled",
                                  "shuffled-wells"])
def test_tiled_sweeps_in_lockstep(name, precision):
    from paper_1705_05784_amd import fams
    s, (wb, pr, vx, _) = _system(name)
    g = fams.Solver(s.row_ptr, s.col, s.val, s.n_matrix, wb, pr, vx, variant=0,
                    precision=precision, n_wells=s.n_wells, smoother=2 if name == "dense" else 1)
    Q = torch.from_numpy(np.random.default_rng(5).standard_normal((32, s.n)))
    one = [g.solve(Q[r], outer="richardson", rtol=0.0, max_iter=1)[0].cpu().numpy()
           for r in range(32)]
    tol = 1e-3 if precision else 1e-10
    for k in (2, 4, 8, 16, 32):   # twice: the second re-uses the published values' state
        for _ in range(2):
            print(f"[lock-step tiles] {name} precision {precision} K {k}", flush=True)
            P = g.solve(Q[:k].contiguous(), outer="richardson", rtol=0.0, max_iter=1)[0].cpu().numpy()
            for r in range(k):
                d = np.abs(P[r] - one[r]).max()
                assert d <= tol * np.abs(one[r]).max(), (k, r, d)
    g.close()
