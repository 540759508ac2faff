"""Neighbour lists: that every pair within reach is listed until the next
rebuild, against the FP64 oracle, which searches all pairs."""
import numpy as np
import pytest

from paper_1711_00336_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    from paper_1711_00336_amd import lbdem
    lbdem.lib()
    return lbdem


@pytest.mark.parametrize("n_dem", [1, 3])
@pytest.mark.parametrize("use_lub", [0, 1])
@pytest.mark.parametrize("shift", [0.0, 6.0])
def test_diagonal_approach_matches_oracle(L, n_dem, use_lub, shift):
    """Two spheres approach along (1, 1, 1) from just outside the list reach
    (d + h_c + 0.1), 0.0149 cells per axis and subcycle: after two subcycles
    0.0298 per axis each, but 0.103 nearer to each other, within reach of the
    lubrication, or in contact without it. In the box and across its periodic
    boundary; one step, every array to 1e-12 of its largest value."""
    from tests.parity_util import compare_states
    from oracle import oracle as O
    p = I.Params(n=(12, 12, 12), periodic=(1, 1, 1), tau=0.6, h_c=0.5, use_lub=use_lub, n_int=10, n_dem=n_dem)
    d = 1.0
    e = np.ones(3) / np.sqrt(3.0)
    gap = 0.5 * (d + (0.5 if use_lub else 0.0) + 0.1 + 1e-4)
    x = np.array([6.0 - gap * e, 6.0 + gap * e]) + shift
    x %= 12.0
    u = np.array([np.full(3, 0.149), np.full(3, -0.149)])
    w = np.array([[1e-3, -2e-3, 5e-4], [-7e-4, 1e-3, 2e-3]])
    parts = I.Particles(x, u, w, np.full(2, d), np.full(2, 200.0))
    o = O.Oracle(p, parts)
    assert o.step(1)["status"] == 0
    apart = O.Oracle(p, I.Particles((x + np.outer([-1.5, 1.5], e)) % 12.0, u, parts.w, parts.d, parts.rho_p))
    apart.step(1)
    assert np.abs(o.state.u - apart.state.u).max() > 1e-3 * np.abs(u).max()  # the pair has acted
    with L.Domain(p) as dom:
        dom.add(parts)
        dom.step(1)
        errs, bad = compare_states(dom.lbdem_get_state(), o.state, p, 1e-12)
    print(f"n_dem {n_dem} lubrication {use_lub} at {x[0]}: {errs}", flush=True)
    assert not bad, errs


def _cluster_and_rest(d):
    """A cluster whose spheres have more neighbours than the lists of a domain
    with the cluster alone hold (56 against 32), and a filling with which they
    hold 64."""
    g = np.stack(np.meshgrid(*[np.arange(5)] * 3, indexing="ij"), -1).reshape(-1, 3)
    cluster = 4.0 + 0.49 * (g - 2)
    g = np.stack(np.meshgrid(*[np.arange(11)] * 3, indexing="ij"), -1).reshape(-1, 3)
    rest = (g + 0.5) * 8.0 / 11.0
    rest = rest[np.linalg.norm(rest[:, None] - cluster[None], axis=-1).min(1) > 0.6]

    def parts(x):
        k = len(x)
        return I.Particles(x, np.zeros((k, 3)), np.zeros((k, 3)), np.full(k, d), np.full(k, 2.5))
    return parts(cluster), parts(rest), parts(np.concatenate([cluster, rest]))


@pytest.mark.parametrize("n_dem", [1, 3])
def test_crowded_spheres_may_be_added_first(L, n_dem):
    """Adding particles judges no list: lists that would overflow with the
    first addition, and not with the second, are built by the first step."""
    from tests.parity_util import compare_states
    from oracle import oracle as O
    p = I.Params(n=(8, 8, 8), periodic=(1, 1, 1), tau=I.SWEEP_TAU, h_c=0.6, n_int=10, n_dem=n_dem)
    cluster, rest, both = _cluster_and_rest(0.48)
    o = O.Oracle(p, both)
    assert o.step(1)["status"] == 0
    with L.Domain(p) as dom:
        dom.add(cluster)
        dom.lbdem_sync()
        dom.add(rest)
        dom.step(1)
        errs, bad = compare_states(dom.lbdem_get_state(), o.state, p, 1e-12)
    print(f"n_dem {n_dem}: {errs}", flush=True)
    assert not bad, errs
    with L.Domain(p) as dom:  # a step on the cluster alone is flagged, as ever
        dom.add(cluster)
        with pytest.raises(L.LbdemError) as e:
            dom.step(1)
        assert e.value.status == L.E_UNSTABLE
