"""The coarse stage alone (no smoother): z = P A_c^{-1} P^T r with the solver's
own P and A_c, at coarse grids whose restriction rows are shorter than a
workgroup, a few thousand entries.  FP64 and the FP32 form
round each product a handful of times: 1e-10 (the inverse's conditioning) and
2e-6 of |P| |A_c^{-1}| |P^T| |r|."""
import numpy as np
import pytest
import scipy.sparse as sp

from workloads import make_small

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("coarse", [(8, 8, 4), (5, 5, 3), (2, 2, 2)])
def test_coarse_stage(coarse, precision):
    from paper_1705_05784_amd import fams
    s = make_small("3d", nx=33, ny=32, nz=17, n_frac=8, len3d=(8, 20))
    wb, pr, vx, _ = fams.full_grid(s, coarse, 4, 4)
    g = fams.Solver(s.row_ptr, s.col, s.val, s.n_matrix, wb, pr, vx, variant=0,
                    precision=precision, smoother=0)
    rp, ci, va = g.prolongation()
    P = sp.csr_matrix((va, ci, rp), shape=(s.n, g.n_coarse))
    Ai = np.linalg.inv(np.asarray(g.coarse_matrix()))
    lens = np.diff(P.tocsc().indptr)
    print(f"[coarse stage] {coarse} precision {precision} row lengths {lens.min()}..{lens.max()}",
          flush=True)
    r = np.random.default_rng(2).standard_normal(s.n)
    z = g.apply_stage(torch.from_numpy(r)).cpu().numpy()
    ref = P @ (Ai @ (P.T @ r))
    bound = abs(P) @ (abs(Ai) @ (abs(P).T @ abs(r)))
    assert (abs(z - ref) <= (2e-6 if precision else 1e-10) * bound.max()).all()
    g.close()
