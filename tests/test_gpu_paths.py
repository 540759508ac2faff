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


def _lattice(n, m, jitter, d_lo, d_hi, rng):
    """m^3 spheres on a jittered cubic lattice of the box n."""
    g = np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing="ij"), -1).reshape(-1, 3) + 0.5
    x = (g + rng.uniform(-jitter, jitter, g.shape) * m / np.min(n)) * (np.asarray(n, float) / m)
    k = rng.permutation(len(x))
    return x[k], rng.uniform(d_lo, d_hi, len(x))


@pytest.mark.parametrize("name,n,m,d,h_c,n_int,n_dem", [
    # lists sorted in place (over 512 entries), eight lanes per particle
    ("long_lists", (10, 10, 10), 20, (0.25, 0.3), 3.0, 2, 1),
    # eight and two lanes per particle, three substeps
    ("lanes8", (15, 15, 15), 14, (0.85, 0.95), 1.0, 10, 3),
    ("lanes2", (40, 38, 39), 36, (0.86, 0.94), 0.9, 4, 3),
    # one lane per particle, more than 64 list entries
    ("lanes1", (48, 48, 48), 52, (0.62, 0.9), 1.7, 2, 1),
])
def test_dem_lane_counts_match_oracle(L, name, n, m, d, h_c, n_int, n_dem):
    """The DEM pass with each number of lanes per particle, with contacts,
    walls and periodic axes, FP64, against the oracle after one step: 1e-12 of
    the largest value (the bar of the other FP64 parity tests). The separate
    force and integration passes give the same bits."""
    from tests.parity_util import compare_states
    from oracle import oracle as O
    rng = np.random.default_rng(11)
    # (far beyond its own diameter the lubrication is not dissipative: kept small)
    tau = 0.5001 if name == "long_lists" else I.SWEEP_TAU
    p = I.Params(n=n, periodic=(1, 1, 0), tau=tau, e_n=0.9, h_c=h_c, n_int=n_int, n_dem=n_dem)
    x, dd = _lattice(n, m, 0.08, d[0], d[1], rng)
    lo, hi = 0.5 * dd, n[2] - 0.5 * dd
    x[:, 2] = np.clip(x[:, 2], lo, hi)
    k = len(x)
    parts = I.Particles(x, rng.normal(size=(k, 3)) * 1e-4, rng.normal(size=(k, 3)) * 1e-4, dd, np.full(k, 2.5))
    print(f"{name}: {k} spheres", flush=True)
    o = O.Oracle(p, parts)
    assert o.step(1)["status"] == 0
    ref = None
    for fuse in (1, 0):
        with L.Domain(p) as dom:
            dom.add(parts)
            dom.lbdem_set_tuning(fuse_substep=fuse)
            dom.step(1)
            st = dom.lbdem_get_state()
        if ref is None:
            ref = st
            errs, bad = compare_states(st, o.state, p, 1e-12)
            print(f"  rel errors {errs}", flush=True)
            assert not bad, errs
        for key in ("df", "x", "u", "w", "a"):
            assert np.array_equal(ref[key], st[key]), key


@pytest.mark.parametrize("k", [1, 63, 64, 65, 129])
@pytest.mark.parametrize("precision,tol", [("fp64", 1e-12), ("fp32dev", 1e-5)])
def test_few_particles_match_oracle(L, k, precision, tol):
    """Particle counts around a wavefront, some overlapping, three substeps."""
    from tests.parity_util import compare_states
    from oracle import oracle as O
    rng = np.random.default_rng(k)
    p = I.Params(n=(12, 13, 14), periodic=(1, 0, 1), tau=0.8, h_c=0.5, n_int=10, n_dem=3, precision=precision)
    d = np.full(k, 0.8)
    x = I.place_spheres(k, p.n, p.periodic, d)
    if k > 1:  # the closest pair overlaps by a hundredth
        far = np.linalg.norm(x[:, None] - x[None], axis=-1) + 9.0 * np.eye(k)
        pair = np.unravel_index(far.argmin(), far.shape)
        d[list(pair)] = 1.01 * far.min()
    parts = I.Particles(x, rng.normal(size=(k, 3)) * 1e-4, rng.normal(size=(k, 3)) * 1e-4, d, np.full(k, 2.5))
    o = O.Oracle(p, parts)
    st0 = o.step(1)
    assert st0["status"] == 0
    with L.Domain(p) as dom:
        dom.add(parts)
        dom.step(1)
        errs, bad = compare_states(dom.lbdem_get_state(), o.state, p, tol)
    print(f"{k} {precision}: {errs}", flush=True)
    assert not bad, errs


@pytest.mark.parametrize("n_int", [2, 3, 10])
@pytest.mark.parametrize("eps,h_c", [(0.05, 0.5), (0.1, 0.5), (0.1, 1.0)])
@pytest.mark.parametrize("precision", ["fp64", "fp32dev"])
def test_lists_built_in_substep_bitwise_equal(L, n_int, eps, h_c, precision):
    """Neighbour lists rebuilt inside the fused pass of one DEM substep (even
    n_int; one, two and eight lanes per particle) and by their own launch:
    heavy spheres that drift by four times the distance of a rebuild."""
    p = I.Params(n=(12, 13, 14), periodic=(1, 1, 1), tau=0.8, h_c=h_c, n_int=n_int, n_dem=1, precision=precision)
    parts = I.make_particles(7, p, I.count_for_fraction(eps, 12 * 13 * 14, 0.5), 0.5, 0.5, 200.0)
    parts.u[:] = (0.03, 0.02, -0.01)
    print(f"{precision} {n_int} {h_c}: {parts.n} spheres", flush=True)
    ref = None
    for fuse in (1, 0):
        with L.Domain(p) as dom:
            dom.add(parts)
            dom.lbdem_set_tuning(fuse_substep=fuse)
            for _ in range(4):
                dom.step(2)
            st = dom.lbdem_get_state()
        if ref is None:
            ref = st
            moved = np.linalg.norm((st["x"] - parts.x + 0.5 * np.array(p.n)) % p.n - 0.5 * np.array(p.n), axis=1)
            assert moved.min() > 4 * 0.05
        for key in ("df", "x", "u", "w", "a"):
            assert np.array_equal(ref[key], st[key]), key


def test_read_out_follows_pending_default_stream_work(L):
    """A read-out into memory that work pending on the default stream still
    writes: the read-out comes last, to device and to pinned host memory."""
    import torch
    p = I.Params(n=(21, 17, 30), periodic=(1, 1, 0), tau=0.8, precision="fp64")
    n = 300
    parts = I.make_particles(2, p, n, 0.5, 0.5, 2.5)
    call = L.lib().lbdem_read_particles
    with L.Domain(p) as dom:
        dom.add(parts)
        dom.step(2)
        want = dom.lbdem_read_particles()
        dev = [torch.empty(n, 3, dtype=torch.float64, device="cuda") for _ in range(4)]
        pin = [torch.empty(n, 3, dtype=torch.float64, pin_memory=True) for _ in range(4)]
        seven = torch.full((n, 3), 7.0, dtype=torch.float64, device="cuda")
        a = torch.randn(8192, 8192, device="cuda")
        b = a @ a
        for mem, out in ((L.MEM_DEVICE, dev), (L.MEM_HOST, pin)):
            torch.cuda.synchronize()
            for _ in range(20):  # a tenth of a second and more
                torch.matmul(a, a, out=b)
            for t in out:
                t.copy_(seven, non_blocking=True)
            assert call(dom.h, mem, *[C.c_void_p(t.data_ptr()) for t in out]) == L.OK
            torch.cuda.synchronize()
            for w, t in zip(want, out):
                same = np.array_equal(w, t.cpu().numpy())
                assert same, mem


@pytest.mark.parametrize("n,precision", [((83, 81, 79), "fp32dev"), ((61, 53, 71), "fp64"), ((61, 53, 11), "fp64"),
                                         ((35, 33, 31), "fp32dev")])
def test_ragged_drag_tiles_bitwise_equal(L, n, precision):
    """Every drag tile where it does not divide the domain (FP32 16x8x8 from
    2^19 cells on and 16x4x4 below, FP64 16x4x8 above 768 small tiles and
    16x4x4 below), halos wrapped on two axes and clamped at the walls of the
    third, against the pass with one thread per particle (variant 3)."""
    p = I.Params(n=n, periodic=(1, 0, 1), tau=0.8, n_int=2, precision=precision)
    rng = np.random.default_rng(n[0])
    k = 3000
    x = rng.random((k, 3)) * np.array(n)
    x[:, 1] = np.clip(x[:, 1], 0.1, n[1] - 0.1)
    x[:100, 0] = n[0] * (1.0 - 1e-9 * rng.random(100))  # last cells of each axis
    x[100:200, 1] = n[1] - 0.1
    x[200:300, 2] = n[2] * (1.0 - 1e-9 * rng.random(100))
    parts = I.Particles(x, rng.normal(size=(k, 3)) * 1e-4, np.zeros((k, 3)), np.full(k, 0.2), np.full(k, 20.0))
    df = I.perturbed_state(3, n[0] * n[1] * n[2], 1e-4)
    ref = None
    for v in (3, 0):
        with L.Domain(p.copy(use_lub=0, T_c=1e3)) as dom:
            dom.lbdem_set_state(df, np.zeros((3, dom.nc)), 0, parts.x, parts.u, parts.w, np.zeros((k, 3)), parts.d,
                                parts.rho_p)
            dom.lbdem_set_gather_variant(v)
            dom.step(1)
            st = dom.lbdem_read_particle_forces()
            st["facc"] = dom.lbdem_read_field(L.FIELD_F_ACC)
            st["x"], st["u"] = dom.lbdem_read_particles()[:2]
        if ref is None:
            ref = st
            assert np.abs(st["F_d"]).max() > 0 and np.abs(st["F_pr"]).max() > 0
        for key in ref:
            same = np.array_equal(ref[key], st[key])
            assert same, (v, key)


@pytest.mark.parametrize("k", [192, 193, 255, 256, 257])
@pytest.mark.parametrize("precision,tol", [("fp64", 1e-12), ("fp32dev", 1e-5)])
def test_single_launch_subcycle_edges(L, k, precision, tol):
    """The substeps of a subcycle in one launch of up to four full wavefronts,
    its last particle count and the first beyond it, against the oracle after
    one step and, bit for bit, against separate force and integration passes."""
    from tests.parity_util import compare_states
    from oracle import oracle as O
    rng = np.random.default_rng(k)
    p = I.Params(n=(16, 13, 14), periodic=(1, 0, 1), tau=0.8, h_c=0.5, n_int=10, n_dem=4, precision=precision)
    d = np.full(k, 0.8)
    x = I.place_spheres(k, p.n, p.periodic, d)
    far = np.linalg.norm(x[:, None] - x[None], axis=-1) + 9.0 * np.eye(k)
    pair = np.unravel_index(far.argmin(), far.shape)
    d[list(pair)] = 1.01 * far.min()  # the closest pair overlaps by a hundredth
    parts = I.Particles(x, rng.normal(size=(k, 3)) * 1e-4, rng.normal(size=(k, 3)) * 1e-4, d, np.full(k, 2.5))
    o = O.Oracle(p, parts)
    assert o.step(1)["status"] == 0
    ref = None
    for fuse in (1, 0):
        with L.Domain(p) as dom:
            dom.add(parts)
            dom.lbdem_set_tuning(fuse_substep=fuse)
            dom.step(1)
            st = dom.lbdem_get_state()
        if ref is None:
            ref = st
            errs, bad = compare_states(st, o.state, p, tol)
            print(f"{k} {precision}: {errs}", flush=True)
            assert not bad, errs
        for key in ("df", "x", "u", "w", "a"):
            assert np.array_equal(ref[key], st[key]), key


@pytest.mark.parametrize("precision,t,tol", [("fp64", 9, 1e-10), ("fp32dev", 11, 1e-5)])
def test_records_beyond_4_gib(L, precision, t, tol):
    """Records that a 32-bit byte offset does not reach (46.7 M spheres of 96 B,
    85 M of 64 B): a periodic box of t^3 copies of a small one steps as the
    small one does. Positions 144 cells out carry 16 times its rounding (3e-14),
    which the gaps (0.05 and more) turn into 1e-12 of a force: 1e-10 of the
    largest velocity; in the FP32 form the rounding of single weights may turn
    over: the bar of its steps."""
    n, m = 16, 40  # 64,000 spheres on a jittered lattice, 15.6 per cell
    rng = np.random.default_rng(4)
    g = np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing="ij"), -1).reshape(-1, 3)
    x = (g + 0.5 + 0.06 * rng.uniform(-1, 1, g.shape)) * (n / m)
    x = np.round(x * 2.0 ** 30) * 2.0 ** -30  # exact in every copy
    k = len(x)
    u = rng.normal(size=(k, 3)) * 1e-4
    small = I.Params(n=(n,) * 3, periodic=(1, 1, 1), tau=I.SWEEP_TAU, h_c=0.1, n_int=2, n_dem=1,
                     precision=precision)
    with L.Domain(small) as dom:
        dom.lbdem_add_particles(x, u, np.zeros((k, 3)), np.full(k, 0.3), np.full(k, 20.0))
        dom.step(1)
        want = dom.lbdem_read_particles()[1]
    assert np.abs(want - u).max() > 1e-2 * np.abs(u).max()
    off = np.stack(np.meshgrid(*[np.arange(t) * float(n)] * 3, indexing="ij"), -1).reshape(-1, 1, 3)
    big = small.copy(n=(n * t,) * 3)
    K = k * t ** 3
    with L.Domain(big) as dom:
        print(f"{K} spheres, {(96 if precision == 'fp64' else 64) * K / 2 ** 30:.2f} GiB of records", flush=True)
        dom.lbdem_add_particles((off + x).reshape(-1, 3), np.tile(u, (t ** 3, 1)), np.zeros((K, 3)), np.full(K, 0.3),
                                np.full(K, 20.0))
        print("added", flush=True)
        dom.step(1)
        print("stepped", flush=True)
        got = np.zeros((K, 3))
        assert L.lib().lbdem_read_particles(dom.h, L.MEM_HOST, None, C.c_void_p(got.ctypes.data), None, None) == L.OK
    err = np.abs(got.reshape(t ** 3, k, 3) - want).max() / np.abs(want).max()
    print(f"largest difference {err}", flush=True)
    assert err < tol


@pytest.mark.parametrize("n", [(7, 3, 9), (3, 8, 5), (6, 5, 3), (3, 3, 3)])
@pytest.mark.parametrize("precision", ["fp64", "fp32dev"])
def test_gathers_on_three_cells_bitwise_equal(L, n, precision):
    """Periodic axes of exactly three cells, whose bins all neighbour every
    cell: each gather variant sums them in the same order. 3.3 spheres per
    cell, so that tiles are staged whole and plane by plane."""
    p = I.Params(n=n, periodic=(1, 1, 1), tau=I.SWEEP_TAU, h_c=0.1, n_int=3, precision=precision)
    rng = np.random.default_rng(5)
    m = int(round((3.3 * np.prod(n)) ** (1 / 3)))
    g = np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing="ij"), -1).reshape(-1, 3)
    x = (g + 0.5 + rng.uniform(-0.2, 0.2, g.shape)) * (np.array(n, float) / m)
    k = len(x)
    parts = I.Particles(x, rng.normal(size=(k, 3)) * 1e-4, np.zeros((k, 3)), rng.uniform(0.2, 0.25, k), np.full(k, 20.0))
    ref = None
    for v in (3, 0, 1, 2, 4):
        with L.Domain(p) as dom:
            dom.lbdem_set_gather_variant(v)
            dom.add(parts)
            dom.step(2)
            st = dom.lbdem_get_state()
            st["facc"] = dom.lbdem_read_field(L.FIELD_F_ACC)
            st["eps"] = dom.lbdem_read_field(L.FIELD_EPS_F)
        if ref is None:
            ref = st
        for key in ref:
            same = np.array_equal(np.asarray(ref[key]), np.asarray(st[key]))
            assert same, (v, key)
