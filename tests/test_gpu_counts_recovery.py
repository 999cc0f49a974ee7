"""The sort's counts, which one paint leaves zero for the next sort, after a
HIP error and under a caller's capture: a paint equals the one of a new
context bit for bit (it sums whole numbers).  The error is the documented one
of a captured run on the default stream."""
import pytest
import torch

from paper_2010_11847_amd import inputs
from paper_2010_11847_amd.binding import PMContext, PMError
from tests.gpu_helpers import banner, to_dev

pytestmark = pytest.mark.gpu


def fail_once(c, w):
    pos, mom = c.pm_init_lpt(3, w.a_list[0])
    c.pm_use_graphs(True)
    with pytest.raises(PMError, match="capture could not start"):
        c.pm_run(w.a_list, pos, mom)
    c.pm_use_graphs(False)
    c.lib.pm_sync(c.ctx)   # takes the error that HIP still holds


@pytest.mark.parametrize("n_mesh,n_p", [(16, 4097), (64, (1 << 17) + 1), (256, (1 << 17) + 1)])
def test_paint_after_an_error(gpu, n_mesh, n_p):
    banner(f"counts after an error n={n_mesh} np={n_p}")
    w = inputs.scaled(inputs.ADJ_SMALL, n_mesh, 16, n_steps=2)
    x = to_dev(inputs.uniform_positions(n_p, n_mesh, seed=n_p))
    want = PMContext(w, max_particles=n_p).pm_paint(x)
    c = PMContext(w, max_particles=n_p)
    fail_once(c, w)
    for _ in range(2):
        assert torch.equal(c.pm_paint(x), want)


@pytest.mark.parametrize("failed", [False, True])
@pytest.mark.parametrize("n_mesh,n_p", [(16, 4097), (128, (1 << 17) + 1)])
def test_captured_paint_and_force(gpu, n_mesh, n_p, failed):
    banner(f"captured paint n={n_mesh} np={n_p} failed={failed}")
    w = inputs.scaled(inputs.ADJ_SMALL, n_mesh, 16, n_steps=2)
    x = to_dev(inputs.uniform_positions(n_p, n_mesh, seed=1))
    y = to_dev(inputs.clustered_positions(n_p, n_mesh, seed=2))
    ref = PMContext(w, max_particles=n_p)
    want = [(ref.pm_paint(p), ref.pm_force(p)) for p in (x, y)]
    c = PMContext(w, max_particles=n_p)
    if failed:
        fail_once(c, w)   # the capture below then records a clear of the counts
    torch.cuda.synchronize()
    s, g, p = torch.cuda.Stream(), torch.cuda.CUDAGraph(), x.clone()
    s.wait_stream(torch.cuda.current_stream())
    c.set_stream(s)
    with torch.cuda.graph(g, stream=s):
        d, f = c.pm_paint(p), c.pm_force(p)
    for i in range(4):
        with torch.cuda.stream(s):
            p.copy_((x, y)[i % 2])
            g.replay()
            if i == 2:   # eager work of the same context between the replays
                e = c.pm_paint(x)
        torch.cuda.synchronize()
        assert torch.equal(d, want[i % 2][0]) and torch.equal(f, want[i % 2][1])
        if i == 2:
            assert torch.equal(e, want[0][0])
