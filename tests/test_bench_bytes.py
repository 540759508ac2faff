"""Byte counts that the benchmark rates launches with (bench.launch_bytes)."""
import importlib.util
import os

import numpy as np
import pytest

from paper_1711_00336_amd import inputs as I

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def bench():
    spec = importlib.util.spec_from_file_location("bench_mod_bytes", os.path.join(ROOT, "bench.py"))
    m = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(m)
    return m


@pytest.mark.parametrize("precision,rec,rs", [("fp32dev", 64, 4), ("fp64", 96, 8)])
@pytest.mark.parametrize("n_dem", [1, 10])
def test_launch_bytes_by_hand(bench, precision, rec, rs, n_dem):
    n, nc, lists = 7, 6 * 5 * 4, 3.0
    p = I.Params(n=(6, 5, 4), precision=precision, n_dem=n_dem)
    z = np.zeros((n, 3))
    case = I.Case("t", p, I.Particles(z, z, z, np.ones(n), np.ones(n)), 0)
    kb = bench.launch_bytes(case, lists, 0, True)
    per = 4 + rec + 3 * 24 + (8 if precision == "fp32dev" else 0) + 24 + rec + 4 * 3
    lone = 24 + 24 + (12 + 9 * rs) + 24
    assert kb["dem_force"] == n * per + (n * lone + nc * 4 * rs if n_dem == 1 else 0)
    assert kb["integrate"] == 0 and kb["nlist"] == 0 and kb["bins"] == 24 * n + 20 * nc
    kb = bench.launch_bytes(case, lists, 0, False)
    assert kb["dem_force"] == n * (4 + rec + 4 * 3 + 48)
    assert kb["integrate"] == n * (6 * 24 + 16 + 24 + 72 + rec)
    # the other classes are those of kernel_bytes
    ref = bench.kernel_bytes(case, lists)
    for k in ("stream_collide", "moments", "cellfields", "part_am", "part_drag", "gather_eps"):
        assert kb[k] == ref[k]
