"""The counts that one sort leaves to the next: whatever ran before on a
context, a paint equals the one of a new context bit for bit (it sums in
whole numbers).  Meshes on both sides of the size from which the keys are
scanned by more than one workgroup (128^3 fills the last one)."""
import pytest
import torch

from paper_2010_11847_amd import inputs
from paper_2010_11847_amd.binding import PMContext
from tests.gpu_helpers import banner, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_mesh,n_part", [(8, 8), (16, 16), (64, 64), (128, 32), (256, 64)])
def test_paint_after_anything_equals_paint_on_a_new_context(gpu, n_mesh, n_part):
    banner(f"sort counts n={n_mesh} np={n_part}")
    w = inputs.scaled(inputs.ADJ_SMALL, n_mesh, n_part, n_steps=2)
    x = [to_dev(inputs.uniform_positions(n_p, n_mesh, seed=n_p)) for n_p in (n_part ** 3, n_part ** 3 // 2 + 1)]
    want = [PMContext(w).pm_paint(p) for p in x]
    c = PMContext(w)

    def same():
        for p, ref in zip(x, want):
            assert torch.equal(c.pm_paint(p), ref)

    same()
    c.pm_force(x[0])
    same()
    pos, mom = c.pm_init_lpt(3, w.a_list[0])
    ck = torch.empty((len(w.a_list), 2, w.n_particles, 3), device="cuda")
    c.pm_run(w.a_list, pos, mom, ckpt=ck)
    same()
    gd = torch.rand((n_mesh,) * 3, device="cuda")
    whole = c.pm_run_adjoint(w.a_list, ck, grad_delta=gd, want_noise_grad=False)
    same()
    # the last point alone: a sort with no paint behind it
    one = c.pm_run_adjoint(w.a_list[-1:], ck[-1:], grad_delta=gd, want_noise_grad=False)
    same()
    assert torch.isfinite(whole[0]).all() and torch.isfinite(one[0]).all()
    c.pm_kdk_step(pos, mom, c.pm_force(pos), w.a_list[0], w.a_list[1])
    same()
