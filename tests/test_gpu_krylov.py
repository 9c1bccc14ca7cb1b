"""GMRES of one right-hand side at the sizes where its orthogonalisation passes
change form: 4, 8, 16 and 32 basis vectors and one more, and restarts over 32.
The oracle is one cycle of the same method in NumPy (the GPU's stage as the
preconditioner, Householder QR for the least squares).  Both minimise the same
residual; its norm relative to ||q|| agrees to a loss of 1e5 roundings of the
first one, 1e-11."""
import numpy as np
import pytest

from tests._cases import small_case

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", ["2d", "3d"])
def test_gmres_cycle_lengths(name):
    from paper_1705_05784_amd import fams
    s, spec = small_case(name)
    wb, pr, vx, _ = fams.full_grid(s, spec["coarse"], spec["d_min"], spec["r_z"])
    g = fams.Solver(s.row_ptr, s.col, s.val, s.n_matrix, wb, pr, vx, variant=0)
    A, q = s.csr(), np.random.default_rng(11).standard_normal(s.n)
    V, Z = [q / np.linalg.norm(q)], []
    for j in range(41):
        Z.append(g.apply_stage(torch.from_numpy(V[-1])).cpu().numpy())
        w = A @ Z[-1]
        for _ in range(2):
            for v in V:
                w = w - (v @ w) * v
        V.append(w / np.linalg.norm(w))
    AZ = np.stack([A @ z for z in Z], axis=1)
    for m in (1, 2, 4, 5, 8, 9, 16, 17, 31, 32, 33, 41):
        print(f"[gmres] {name} restart {m}", flush=True)
        p, info = g.solve(torch.from_numpy(q), outer="gmres", restart=m, rtol=1e-30, max_iter=m)
        y = np.linalg.lstsq(AZ[:, :m], q, rcond=None)[0]
        ref = np.linalg.norm(q - AZ[:, :m] @ y) / np.linalg.norm(q)
        got = np.linalg.norm(q - A @ p.cpu().numpy()) / np.linalg.norm(q)
        assert info[0]["iterations"] == m
        assert abs(got - ref) <= 1e-11, (m, got, ref)
    g.close()
