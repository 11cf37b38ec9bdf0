"""The march's 64-bit cell index, which grids above 1625^3 take, and the
deposits of grids whose lines of Gamma do not fit the table's 32-bit keys
(3251^3 and more: more memory than a card has), on small grids: a second build
of the library takes the 64-bit index on every grid and the table only below
1000 lines (19^3).  Against the oracle under the bars of the 32-bit index:
counts equal, FP64 within 1e-11 (a cell takes at most a few 10^4 deposits here,
each within a few ulp; 1e-10 through a spectrum's table), the mixed path within
the method's 1e-4."""
import importlib.util
import os

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def edges(gpu):
    """The binding on the second build, as a module of its own."""
    spec = importlib.util.spec_from_file_location("nyxrt_edges", gpu.__file__)
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    mod.LIB_PATH = os.path.join(os.path.dirname(gpu.__file__), "libnyxrt_edges.so")
    mod.load()
    return mod


@pytest.mark.parametrize("n", [3, 8, 17, 19, 20, 24])
@pytest.mark.parametrize("periodic", [True, False])
@pytest.mark.parametrize("corr,spectrum", [(0, 0), (2, 0), (4, 0), (2, 1)])
def test_wide_index(edges, orc, n, periodic, corr, spectrum):
    g = np.random.default_rng(900 + 10 * n + periodic)
    nH = 1e-3 * np.exp(g.standard_normal((n, n, n)))
    x = np.where(g.random((n, n, n)) < 0.3, 1.0 - 1e-4, 0.0)
    pos = np.array([[0.3, 0.6, 0.9], [0.5, 0.5, 0.5], [0.0, 0.0, 0.0], [n - 0.5, 0.0, 0.25]])
    ndot = W.lognormal_values(4, 1e50, 1.0, g)
    h = 0.1 / (W.SIGMA0 * 1e-3)
    kw = dict(periodic=periodic, n_min_ray=64.0 if n < 9 else 4.0, l_max=6, tau_max=30.0,
              n_th=4e-4, corr=corr, spectrum=spectrum, spec_param=5e4 if spectrum else 0.0)
    ref, rb = orc.trace(orc.make_params(n, h, **kw), nH, x, pos, ndot)
    for prec, tol in ((0, 1e-10 if spectrum else 1e-11), (1, 1e-4)):
        ctx = edges.init_grid(edges.make_desc(n, h, precision=prec, **kw), nH, x, device="cuda:0",
                              max_sources=4, ray_capacity=1 << 18)
        ctx.add_sources(pos, ndot)
        gamma, b = ctx.trace_step()
        got = gamma.cpu().numpy()
        ctx.destroy()
        for k in ("segments", "rays", "splits"):
            assert b[k] == rb[k], (prec, k)
        mask = ref > 1e-6 * ref.max()
        assert np.abs(got[mask] / ref[mask] - 1).max() <= tol, prec
        for k in ("absorbed", "escaped", "truncated"):
            assert abs(b[k] - rb[k]) <= (1e-10 if prec == 0 else 1e-6) * rb["emitted"], (prec, k)


@pytest.mark.parametrize("prec", [0, 1])
def test_segment_counts_added_early(edges, orc, prec):
    """A lane's 32-bit count of segments is added to the pass's 64-bit one before
    it can wrap (2^31; 50 in the second build): the count is the oracle's, in
    runs of 64 that make every wavefront claim often."""
    n = 24
    g = np.random.default_rng(17)
    nH = 1e-3 * np.exp(g.standard_normal((n, n, n)))
    x = np.full((n, n, n), 0.9)
    pos, ndot = W.uniform_positions(12, n, g), W.lognormal_values(12, 1e50, 1.0, g)
    h = 0.1 / (W.SIGMA0 * 1e-3)
    kw = dict(periodic=True, n_min_ray=4.0, l_max=6, tau_max=30.0)
    _, rb = orc.trace(orc.make_params(n, h, **kw), nH, x, pos, ndot)
    ctx = edges.init_grid(edges.make_desc(n, h, precision=prec, **kw), nH, x, device="cuda:0",
                          max_sources=12, ray_capacity=1 << 20)
    ctx.add_sources(pos, ndot)
    for refill, bpc in ((0, 0), (1, 1), (64, 1)):
        ctx.set_tuning(refill_min=refill, claim=64 if bpc else 0, blocks_per_cu=bpc)
        _, b = ctx.trace_step()
        assert b["segments"] == rb["segments"] > 50 * rb["rays"] / 64
    ctx.destroy()
