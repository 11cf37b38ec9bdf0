"""Grids and rays at the edges of the march's fast path, against the oracle.

Boxes of one to a few cells, where every cell lies on the boundary layer and
wraps or leaves are decided from the box planes, next to boxes with the first
interior cells; and rays that reach the levels whose deposits are summed in
FP64 in the mixed path.  FP64 paths take the oracle's decisions exactly, so
the counts are equal and Gamma agrees to the rounding of its sums: a cell takes
at most a few 10^4 deposits here, each within a few ulp (1e-16), so 1e-11
bounds the FP64 path; the mixed path's bar is the method's 1e-4."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 8, 9, 17])
@pytest.mark.parametrize("periodic", [True, False])
@pytest.mark.parametrize("corr", [2, 4])
def test_tiny_boxes(gpu, orc, n, periodic, corr):
    g = np.random.default_rng(700 + 10 * n + periodic)
    nH = 1e-3 * np.exp(g.standard_normal((n, n, n)))
    x = np.where(g.random((n, n, n)) < 0.3, 1.0 - 1e-4, 0.0)
    # inside a cell, on its centre, and on the box's planes and corner
    pos = np.array([[0.3, 0.6, 0.9], [0.5, 0.5, 0.5], [0.0, 0.0, 0.0], [n - 0.5, 0.0, 0.25]])
    ndot = W.lognormal_values(4, 1e50, 1.0, g)
    h = 0.1 / (W.SIGMA0 * 1e-3)  # thin enough for rays to cross the box and split
    kw = dict(periodic=periodic, n_min_ray=64.0 if n < 9 else 4.0, l_max=7, tau_max=30.0,
              n_th=4e-4, corr=corr)
    ref, rb = orc.trace(orc.make_params(n, h, **kw), nH, x, pos, ndot)
    if n == 17:
        assert rb["rays_per_level"][5] > 0  # FP64 sums in the mixed path too
    for prec, tol in ((0, 1e-11), (1, 1e-4)):
        ctx = gpu.init_grid(gpu.make_desc(n, h, precision=prec, **kw), nH, x, device="cuda:0",
                            max_sources=4, ray_capacity=1 << 18)
        ctx.add_sources(pos, ndot)
        gamma, b = ctx.trace_step()
        got = gamma.cpu().numpy()
        ctx.destroy()
        for k in ("segments", "rays", "splits"):
            assert b[k] == rb[k], (prec, k)
        assert b["rays_per_level"] == rb["rays_per_level"][:15]
        mask = ref > 1e-6 * ref.max()
        assert np.abs(got[mask] / ref[mask] - 1).max() <= tol, prec
        for k in ("absorbed", "escaped", "truncated"):
            assert abs(b[k] - rb[k]) <= (1e-10 if prec == 0 else 1e-6) * rb["emitted"], (prec, k)


@pytest.mark.parametrize("n,l_max", [(4, 0), (4, 1), (4, 9), (4, 10), (128, 11)])
def test_direction_table_levels(gpu, orc, n, l_max):
    """The direction table formed on the device (its azimuths fit the scratch
    space) and the one formed on the host (4^3 with levels past 9) hold the
    oracle's directions bit for bit at every level."""
    import torch
    one = torch.ones((n, n, n), dtype=torch.float64, device="cuda:0")
    ctx = gpu.init_grid(gpu.make_desc(n, 1e20, l_max=l_max), one, 0 * one, device="cuda:0",
                        max_sources=1, ray_capacity=4096)
    g = np.random.default_rng(5)
    for level in range(l_max + 1):
        npix = 12 * 4 ** level
        for first in {0, max(0, npix - 40), npix // 2, *g.integers(0, npix, 12).tolist()}:
            count = min(40, npix - first)
            ref = np.array([orc.pix2vec_nest(level, p) for p in range(first, first + count)])
            np.testing.assert_array_equal(ctx.healpix_dirs(level, first, count), ref,
                                          err_msg=str((level, first)))
    ctx.destroy()
