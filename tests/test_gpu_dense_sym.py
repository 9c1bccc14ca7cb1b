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


@pytest.mark.parametrize("n", [1100, 2500])
def test_symmetric_form_is_as_exact(n):
    """The symmetric form's residual is no larger than the full form's, which a
    matrix 1e-13 away takes (its own residual), at condition 1e6."""
    from paper_1705_05784_amd import fams
    print(f"[dense] exactness n={n}", flush=True)
    rng = np.random.default_rng(n)
    q, _ = np.linalg.qr(rng.standard_normal((n, n)))
    a = (q * np.logspace(0, -6, n)) @ q.T
    a = (a + a.T) / 2
    d = np.sqrt(np.diag(a))
    b = a + np.triu(1e-13 * np.outer(d, d) * rng.choice((-1.0, 1.0), (n, n)), 1)
    e = []
    for m in (a, b):
        x = fams.dense_op(1, m).cpu().numpy()
        e.append(np.linalg.norm(x @ m - np.eye(n)))
    assert e[0] <= e[1], e
