"""Growth factors after other calls on the same context: the growth ODE's
trajectory is kept with a context, so whatever was asked before, and in which
order, a factor is the one of a new context, and the oracle's."""
import pytest

from oracle import cosmology as Cm
from paper_2010_11847_amd import inputs
from paper_2010_11847_amd.binding import PMContext
from tests.gpu_helpers import banner

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", [1, -1])
def test_growth_factors_do_not_depend_on_earlier_calls(gpu, order):
    banner(f"growth calls order={order}")
    w = inputs.scaled(inputs.MEDIUM, 16, 16)
    c = PMContext(w)
    for a in [1e-5, 2e-3, 0.1, 0.3333, 0.999, 1.0, 1.25][::order]:
        got = c.pm_growth(a)
        c.pm_kdk_factors([0.5 * a, a])
        assert got == PMContext(w).pm_growth(a)
        if a > 1e-5:
            for v, o in zip(("D1", "f1", "D2", "f2"), Cm.growth(a, w.cosmo.omega_m)):
                assert abs(got[v] / float(o[0]) - 1) < 1e-9
    k = c.pm_kdk_factors(w.a_list)
    for x, y in zip(k, PMContext(w).pm_kdk_factors(w.a_list)):
        assert (x == y).all()
