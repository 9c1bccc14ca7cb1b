"""A sweep that gave up is reported, whichever handle it ran on, and the next
call starts anew.  The word that a bounded wait sets on giving up is set here
from outside (the allocator hook serves the two-int buffers from tensors that
the test holds): every wait of the sweeps then gives up at its first look, all
kernels end as always, and the step must report FAMS_ERR_DEVICE once."""
import numpy as np
import pytest

from tests._cases import small_case

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEVICE = -7


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("which", ["own", "per-medium"])
def test_given_up_wait_is_reported(which, precision):
    from paper_1705_05784_amd import fams
    words, live = {}, []

    def alloc(ctx, nbytes, stream):
        if nbytes == 8:
            t = torch.zeros(64, dtype=torch.int32, device="cuda")
            words[t.data_ptr()] = t
            live.append(t.data_ptr())
            return t.data_ptr()
        return torch.cuda.caching_allocator_alloc(int(nbytes), torch.cuda.current_device(),
                                                  int(stream or 0))

    def free(ctx, ptr, stream):
        if ptr in words:
            if ptr in live:
                live.remove(ptr)
            return
        torch.cuda.caching_allocator_delete(int(ptr))

    hook = fams.AllocatorHook(None, fams._ALLOC_FN(alloc), fams._FREE_FN(free))
    s, spec = small_case("3d")
    wb, pr, vx, _ = fams.full_grid(s, spec["coarse"], spec["d_min"], spec["r_z"])
    g = fams.Solver(s.row_ptr, s.col, s.val, s.n_matrix, wb, pr, vx, precision=precision,
                    smoother=2, allocator=hook)
    assert len(live) == 2   # the handle's error words, then the per-medium stage's
    word = words[live[which == "per-medium"]]
    print(f"[sweep errors] {which} precision {precision}", flush=True)
    r = torch.from_numpy(np.random.default_rng(5).standard_normal(s.n)).cuda()
    Q = torch.stack([r, 2.0 * r])
    once = dict(outer="richardson", rtol=0.0, max_iter=1)
    z = g.apply_stage(r).cpu().numpy()
    P = g.solve(Q, **once)[0].cpu().numpy()
    word[0] = 2
    torch.cuda.synchronize()
    with pytest.raises(fams.FamsError) as e:
        g.apply_stage(r)
    assert e.value.status == DEVICE, e.value
    assert np.array_equal(g.apply_stage(r).cpu().numpy(), z)
    assert np.array_equal(g.solve(Q, **once)[0].cpu().numpy(), P)
    assert np.array_equal(g.apply_stage(r).cpu().numpy(), z)
    g.close()
