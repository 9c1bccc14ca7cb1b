"""A solve whose buffers are refused: whatever allocation of a handle's first
solve an allocator hook refuses, the solve either goes on with less or reports
FAMS_ERR_OOM, and the solve after it has every buffer it needs.  The results
are those of a handle that was refused nothing: the second solve's the same
bits, the first one's (narrower groups, other sweeps) to 1e-10 in FP64 and 1e-3
with the FP32 stage, the bounds of the lock-step solves against single ones."""
import numpy as np
import pytest

from tests._cases import small_case

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

OOM = -6
ONCE = dict(outer="gmres", restart=4, rtol=0.0, max_iter=3)


class Hook:
    """torch's caching allocator, with a rule for what is refused."""

    def __init__(self):
        from paper_1705_05784_amd import fams
        self.sizes, self.rule = [], None

        def alloc(ctx, nbytes, stream):
            self.sizes.append(int(nbytes))
            if self.rule and self.rule(len(self.sizes) - 1, int(nbytes)):
                return None
            return torch.cuda.caching_allocator_alloc(int(nbytes), torch.cuda.current_device(),
                                                      int(stream or 0))

        def free(ctx, ptr, stream):
            torch.cuda.caching_allocator_delete(int(ptr))
        self.c = fams.AllocatorHook(None, fams._ALLOC_FN(alloc), fams._FREE_FN(free))

    def arm(self, rule):
        self.sizes, self.rule = [], rule


def _solver(hook, smoother=1, precision=0):
    from paper_1705_05784_amd import fams
    s, spec = small_case("3d")
    wb, pr, vx, _ = fams.full_grid(s, spec["coarse"], spec["d_min"], spec["r_z"])
    return fams.Solver(s.row_ptr, s.col, s.val, s.n_matrix, wb, pr, vx, variant=0, alpha=1e-2,
                       precision=precision, smoother=smoother, allocator=hook.c)


def _rhs(n, k):
    q = torch.from_numpy(np.random.default_rng(k).standard_normal((k, n)))
    return (q if k > 1 else q[0]).cuda()


def _refuse_each(nrhs, smoother=1, precision=0, rule=None, most=None):
    """The first solve of a new handle with its k-th allocation refused, for
    every k (or with what `rule(k)` refuses), then a second one with nothing
    refused; returns how many first solves went through."""
    from paper_1705_05784_amd import fams
    hook = Hook()
    g = _solver(hook, smoother, precision)
    q = _rhs(g.n, nrhs)
    hook.arm(None)
    ref = g.solve(q, **ONCE)[0].cpu().numpy()
    count = len(hook.sizes)
    g.close()
    assert count > 0
    through = 0
    for k in range(min(count, most or count)):
        print(f"[refusals] nrhs {nrhs} smoother {smoother} precision {precision} refused {k}",
              flush=True)
        hook.arm(None)
        g = _solver(hook, smoother, precision)
        hook.arm(rule(k) if rule else lambda i, nbytes: i == k)
        try:
            p = g.solve(q, **ONCE)[0].cpu().numpy()
            assert np.abs(p - ref).max() <= (1e-3 if precision else 1e-10) * np.abs(ref).max()
            through += 1
        except fams.FamsError as e:
            assert e.status == OOM, e
        hook.arm(None)
        assert np.array_equal(g.solve(q, **ONCE)[0].cpu().numpy(), ref), k
        g.close()
    return through


@pytest.mark.parametrize("precision", [0, 1])
def test_single_solve(precision):
    assert _refuse_each(1, precision=precision) == 0


def test_fixed_width_matrices():
    """Lock-step solves: the overflow table of A, then of P (two ints a row)."""
    hook = Hook()
    g = _solver(hook)
    n = g.n
    g.close()

    def rule(k):
        seen = [0]

        def refuse(i, nbytes):
            seen[0] += nbytes == 8 * n
            return nbytes == 8 * n and seen[0] == k % 2 + 1
        return refuse
    assert _refuse_each(4, rule=rule, most=2) == 0


@pytest.mark.parametrize("smoother,precision", [(1, 0), (1, 1), (2, 0)])
def test_lockstep_solve(smoother, precision):
    """Each allocation by itself: groups narrow and the solve goes on where
    the work space and the sweeps' part of the schedule are concerned."""
    assert _refuse_each(7, smoother, precision) > 10


@pytest.mark.parametrize("smoother,precision", [(1, 0), (1, 1), (2, 0)])
def test_lockstep_solve_without_room(smoother, precision):
    """Everything from the k-th allocation on: no first solve has room."""
    assert _refuse_each(4, smoother, precision, lambda k: lambda i, nbytes: i >= k) == 0


@pytest.mark.parametrize("smoother,precision", [(1, 0), (1, 1), (2, 0)])
def test_pair_without_records(smoother, precision):
    """A pair of right-hand sides goes on without the tiles' records (48 to
    128 bytes a row): the sweeps take the level chunks then, as they do where
    the block vectors pass 4 GiB."""
    hook = Hook()
    g = _solver(hook, smoother, precision)
    q = _rhs(g.n, 2)
    ref = g.solve(q, **ONCE)[0].cpu().numpy()
    g.close()
    hook = Hook()
    g = _solver(hook, smoother, precision)
    refused = []

    def rule(i, nbytes):   # the second of the two arrays, allocated one after the other
        if 48 * g.n <= nbytes <= 128 * g.n and hook.sizes[-2:] == [nbytes, nbytes]:
            refused.append(nbytes)
            return True
        return False
    hook.arm(rule)
    for k in range(2):
        p = g.solve(q, **ONCE)[0].cpu().numpy()
        assert np.abs(p - ref).max() <= (1e-3 if precision else 1e-10) * np.abs(ref).max()
        assert len(refused) == k + 1
    hook.arm(None)
    assert np.array_equal(g.solve(q, **ONCE)[0].cpu().numpy(), ref)
    g.close()
