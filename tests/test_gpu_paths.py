"""Launch paths that a domain's size, density or precision selects, each
against the general path or the FP64 oracle."""
import ctypes as C

import numpy as np
import pytest

from paper_1711_00336_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    from paper_1711_00336_amd import lbdem
    lbdem.lib()
    return lbdem


@pytest.mark.parametrize("eps,d", [(0.16, 0.5), (0.3, 0.5), (0.2, 0.3)])
@pytest.mark.parametrize("precision", ["fp64", "fp32dev"])
def test_crowded_gather_tiles_bitwise_equal(L, eps, d, precision):
    """Tiles whose halo exceeds the staging buffer: staged in runs of planes
    (2.4 and 4.6 spheres per cell: several planes, one plane per run), or per
    cell where one plane exceeds it (14 per cell). Ragged edges on every
    axis; the per-cell gather (variant 3) is the general path."""
    n = (18, 17, 19)
    p = I.Params(n=n, periodic=(1, 1, 0), tau=I.SWEEP_TAU, h_c=d, n_int=3, precision=precision)
    parts = I.make_particles(5, p, I.count_for_fraction(eps, n[0] * n[1] * n[2], d), d, d, 2.5)
    print(f"{precision}: {parts.n} spheres", flush=True)
    ref = None
    for v in (3, 0, 1, 2, 4):
        with L.Domain(p) as dom:
            dom.add(parts)
            dom.lbdem_set_gather_variant(v)
            dom.step(1)
            st = dom.lbdem_get_state()
            st["facc"] = dom.lbdem_read_field(L.FIELD_F_ACC)
            st["eps"] = dom.lbdem_read_field(L.FIELD_EPS_F)
        if ref is None:
            ref = st
        for k in ref:
            assert np.array_equal(np.asarray(ref[k]), np.asarray(st[k])), (v, k)


@pytest.mark.parametrize("n", [1, 255, 257, 1000])
def test_particle_read_out_orders(L, n):
    """Read-outs return insertion order, whatever the slot order, to host and
    to device memory."""
    import torch
    p = I.Params(n=(21, 17, 30), periodic=(1, 1, 0), tau=0.8, precision="fp64")
    parts = I.make_particles(2, p, n, 0.5, 0.5, 2.5)
    rng = np.random.default_rng(n)
    parts.u[:] = rng.normal(size=(n, 3)) * 1e-4
    parts.w[:] = rng.normal(size=(n, 3)) * 1e-4
    parts.d[:] = 0.5 - 0.1 * rng.random(n)
    parts.rho_p[:] = 2.0 + rng.random(n)
    with L.Domain(p) as dom:
        dom.add(parts)
        st = dom.lbdem_get_state()
        for k, v in dict(x=parts.x, u=parts.u, w=parts.w, d=parts.d, rho_p=parts.rho_p).items():
            assert np.array_equal(st[k], v), k
        dom.step(2)
        host = dom.lbdem_read_particles()
        dev = [torch.zeros(n, 3, dtype=torch.float64, device="cuda") for _ in range(4)]
        torch.cuda.synchronize()
        ptr = [C.c_void_p(t.data_ptr()) for t in dev]
        assert L.lib().lbdem_read_particles(dom.h, L.MEM_DEVICE, *ptr) == L.OK
        for a, b in zip(host, dev):
            assert np.array_equal(a, b.cpu().numpy())
        only_w = np.zeros((n, 3))
        assert L.lib().lbdem_read_particles(dom.h, L.MEM_HOST, None, None, C.c_void_p(only_w.ctypes.data), None) == L.OK
        assert np.array_equal(only_w, host[2])
