"""The coarse inverse over one block of 1024 columns: a symmetric matrix takes
the form that keeps the lower triangle only, any other (with positive pivots)
the full one.  x a = I to 1e-10, as for the smaller sizes."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sym", [True, False])
@pytest.mark.parametrize("n", [1025, 1056, 1801, 2048, 3105])
def test_block_inverse(n, sym):
    from paper_1705_05784_amd import fams
    print(f"[dense] block inverse n={n} sym={sym}", flush=True)
    m = np.random.default_rng(n).standard_normal((n, n)) / np.sqrt(n)
    a = m @ m.T + np.eye(n) if sym else 0.25 * m + 2.0 * np.eye(n)
    x = fams.dense_op(1, a).cpu().numpy()
    assert np.abs(x @ a - np.eye(n)).max() <= 1e-10
    assert np.array_equal(x, x.T) == sym
