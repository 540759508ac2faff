"""The diagnostics' sums do not depend on where the particles lie: a domain
that has run (slots as its lists left them), the same state loaded afresh, and
every launch choice give the same bits."""
import numpy as np
import pytest

from paper_1711_00336_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    from paper_1711_00336_amd import lbdem
    lbdem.lib()
    return lbdem


def _same(a, b):
    for k in a:
        assert np.array_equal(np.asarray(a[k]), np.asarray(b[k])), (k, a[k], b[k])


@pytest.mark.parametrize("n_dem", [1, 3])
@pytest.mark.parametrize("precision", ["fp64", "fp32dev"])
def test_diagnostics_do_not_depend_on_the_slots(L, precision, n_dem):
    p = I.Params(n=(40, 37, 35), periodic=(1, 1, 1), tau=0.6, n_int=10, n_dem=n_dem, precision=precision)
    parts = I.make_particles(3, p, I.count_for_fraction(0.08, 40 * 37 * 35, 0.7), 0.6, 0.8, 200.0)
    rng = np.random.default_rng(1)
    parts.u[:] = rng.normal(size=parts.u.shape) * 0.01
    print(f"{precision} {n_dem}: {parts.n} spheres", flush=True)
    ref = None
    for order, block in ((-1, 32), (1, 16), (0, 32), (1, 7)):
        with L.Domain(p) as dom:
            dom.add(parts)
            dom.lbdem_set_tuning(dem_order=order, dem_block=(block,) * 3)
            dom.step(4)
            d = dom.lbdem_diagnostics()
            _same(d, dom.lbdem_diagnostics_noalloc())
            st = dom.lbdem_get_state()
        if ref is None:
            ref = d
            with L.Domain(p) as dom:
                dom.lbdem_set_state(st["df"], st["uprev"], st["step"], st["x"], st["u"], st["w"], st["a"], st["d"],
                                    st["rho_p"])
                _same(ref, dom.lbdem_diagnostics())
        _same(ref, d)
