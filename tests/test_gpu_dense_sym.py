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


@pytest.mark.parametrize("off", [1e-6, 1e-9, 1e-12, 1e-13])
def test_slightly_asymmetric(off):
    """A matrix that is not quite symmetric is inverted as given, not the one of
    its lower triangle: x a = I to the same 1e-10."""
    from paper_1705_05784_amd import fams
    n = 1801
    print(f"[dense] asymmetry {off:g}", flush=True)
    rng = np.random.default_rng(n)
    m = rng.standard_normal((n, n)) / np.sqrt(n)
    a = m @ m.T + np.eye(n)
    d = np.sqrt(np.diag(a))
    a += np.triu(off * np.outer(d, d) * rng.choice((-1.0, 1.0), (n, n)), 1)
    x = fams.dense_op(1, a).cpu().numpy()
    assert np.abs(x @ a - np.eye(n)).max() <= 1e-10
    assert not np.array_equal(x, x.T)
