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


def test_direction_table_windows(gpu, orc):
    """Levels to 11 on a 4^3 grid: the azimuths pass through the scratch space
    (2^18 of them at a time) in eight windows.  The pixels on both sides of
    every window's ends, from the oracle; and the table takes the device's
    time, not the host's, which is hundreds of times level 9's (16 times the
    pixels and 8 passes over them: bounded by 60 times)."""
    import time

    import torch
    one = torch.ones((4, 4, 4), dtype=torch.float64, device="cuda:0")

    def init(l_max):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        ctx = gpu.init_grid(gpu.make_desc(4, 1e20, l_max=l_max), one, 0 * one, device="cuda:0",
                            max_sources=1, ray_capacity=4096)
        torch.cuda.synchronize()
        return ctx, time.perf_counter() - t0

    level, ns = 11, 1 << 11
    ctx, _ = init(level)
    # azimuth index -> ring nr and step k of the north cap, whose pixels lie at
    # the odd steps: one of each pair of neighbours is a pixel's
    for edge in [w << 18 for w in range(1, 8)]:
        for i in (edge - 1, edge):
            nr = int(1.5 + np.sqrt(2.0 * i + 0.25))
            while (nr - 1) * (nr - 2) // 2 > i:
                nr -= 1
            k = i - (nr - 1) * (nr - 2) // 2 + 1
            # face 0 (jpll 1): num = nr + ix - iy = k, ring 2 ns - ix - iy - 1 = nr
            if k % 2 == 0:
                continue
            d, t = k - nr, 2 * ns - 1 - nr
            ix, iy = (t + d) // 2, (t - d) // 2
            pix = sum(((ix >> b) & 1) << (2 * b) | ((iy >> b) & 1) << (2 * b + 1)
                      for b in range(11))
            np.testing.assert_array_equal(ctx.healpix_dirs(level, pix, 1)[0],
                                          orc.pix2vec_nest(level, pix), err_msg=str((nr, k)))
    g = np.random.default_rng(3)
    for pix in g.integers(0, 12 * 4 ** level, 300).tolist():
        np.testing.assert_array_equal(ctx.healpix_dirs(level, pix, 1)[0],
                                      orc.pix2vec_nest(level, pix), err_msg=str(pix))
    ctx.destroy()
    times = {}
    for l_max in (9, 11, 9, 11):
        ctx, t = init(l_max)
        ctx.destroy()
        times[l_max] = min(t, times.get(l_max, np.inf))
    assert times[11] < 60 * times[9], times


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("m", [5, 2731, 21845, 21846, 43690, 43691, 65536, 65537, 87381, 87382])
def test_first_runs(gpu, m, prec):
    """Launches whose rays the first runs just cover or just do not (12 m rays
    at level 0: 64, 128, 192 and 256 for each of 4096 wavefronts): every ray is
    marched once whatever the run sizes, so the counts agree with fixed runs of
    128, and each term of the budget to the rounding of its sums."""
    n = 32
    g = np.random.default_rng(m)
    x = np.where(g.random((n, n, n)) < 0.3, 1.0 - 1e-4, 0.0)
    nH = 1e-3 * np.exp(g.standard_normal((n, n, n)))
    pos = W.uniform_positions(m, n, g)
    ndot = W.lognormal_values(m, 1e50, 1.0, g)
    h = 2.0 / (W.SIGMA0 * 1e-3)  # rays stop in both ways
    ctx = gpu.init_grid(gpu.make_desc(n, h, periodic=False, n_min_ray=4.0, l_max=1,
                                      precision=prec), nH, x, device="cuda:0", max_sources=m,
                        ray_capacity=1 << 22)
    ctx.add_sources(pos, ndot)
    ctx.set_tuning(refill_min=16, claim=128, graph=1)
    _, ref = ctx.trace_step()
    assert ref["rays_per_level"][0] == 12 * m and ref["truncated"] > 0 and ref["escaped"] > 0
    for graph in (1, 2):
        ctx.set_tuning(graph=graph)
        _, b = ctx.trace_step()
        assert [b[k] for k in ("segments", "rays", "splits", "rays_per_level")] == [
            ref[k] for k in ("segments", "rays", "splits", "rays_per_level")]
        for k in ("absorbed", "escaped", "truncated"):
            assert abs(b[k] - ref[k]) <= (1e-10 if prec == 0 else 1e-6) * ref["emitted"], k
    ctx.destroy()


@pytest.mark.parametrize("periodic", [True, False])
@pytest.mark.parametrize("kw", [dict(n_min_ray=0.0, l_max=7), dict(n_min_ray=0.05, l_max=4)])
def test_mixed_sums_of_the_first_levels(gpu, orc, periodic, kw):
    """Mixed passes whose long rays never reach the levels that are summed in
    FP64: every deposit is summed in FP32 slots, within the method's 1e-4."""
    n = 48
    g = np.random.default_rng(21 + periodic)
    nH = 1e-3 * np.exp(g.standard_normal((n, n, n)))
    x = np.where(g.random((n, n, n)) < 0.5, 1.0 - 1e-4, 0.9)
    pos, ndot = W.uniform_positions(200, n, g), W.lognormal_values(200, 1e50, 1.0, g)
    h = 0.2 / (W.SIGMA0 * 1e-3)
    kw = dict(periodic=periodic, tau_max=30.0, n_th=4e-4, **kw)
    ref, rb = orc.trace(orc.make_params(n, h, **kw), nH, x, pos, ndot)
    assert rb["segments"] > 10 * rb["rays"] and sum(rb["rays_per_level"][5:]) == 0
    ctx = gpu.init_grid(gpu.make_desc(n, h, precision=1, **kw), nH, x, device="cuda:0",
                        max_sources=200, ray_capacity=1 << 20)
    ctx.add_sources(pos, ndot)
    gamma, b = ctx.trace_step()
    got = gamma.cpu().numpy()
    ctx.destroy()
    for k in ("segments", "rays", "splits"):
        assert b[k] == rb[k], k
    mask = ref > 1e-6 * ref.max()
    assert np.abs(got[mask] / ref[mask] - 1).max() <= 1e-4
    for k in ("absorbed", "escaped", "truncated"):
        assert abs(b[k] - rb[k]) <= 1e-6 * rb["emitted"], k
