"""Sizes at which the merge's kernels change their work, against the oracle:
catalogues around the sort's tile and its powers of two, groups around a
wavefront's 64 members, and radii and boxes on both sides of the near-shell
bitmap's reach (radii to 14.5 cells, boxes of 31 cells and more; past them the
hash table).  The catalogue is integer work and must match exactly; rates are
summed in the same order on both sides (1e-13)."""
import numpy as np
import pytest

import workloads as W
from test_gpu_merge import check_same, gpu_merge

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [1, 2, 3, 63, 65, 2047, 2048, 2049, 4097, 9000])
def test_sort_sizes(gpu, orc, m):
    n = 48
    g = np.random.default_rng(m)
    pos = W.uniform_positions(m, n, g)
    ndot = W.lognormal_values(m, 1e50, 2.0, g)
    x = np.where(g.random((n, n, n)) < 0.5, 0.95, 0.0)
    kw = dict(dr=1.0, r_max=2.0, f_req=0.3)
    ref = orc.merge_sources(orc.make_merge_params(**kw), n, True, x, pos, ndot)
    check_same(ref, gpu_merge(gpu, n, True, x, pos, ndot, gpu.make_merge_params(**kw)))


@pytest.mark.parametrize("members", [2, 63, 64, 65, 200])
@pytest.mark.parametrize("periodic", [True, False])
def test_group_sizes(gpu, orc, members, periodic):
    """Ionized everywhere: every source has the largest radius, and the ones
    around one corner of the box form one group (across its faces if periodic)."""
    n = 64
    g = np.random.default_rng(members)
    offsets = g.permutation(13 ** 3)[:members]
    cell = np.stack([offsets % 13, offsets // 13 % 13, offsets // 169], 1) + (n - 6 if periodic
                                                                            else 3)
    pos = cell % n + 0.5
    ndot = W.lognormal_values(members, 1e50, 2.0, g)
    x = np.full((n, n, n), 0.99)
    ref = orc.merge_sources(orc.make_merge_params(), n, periodic, x, pos, ndot)
    got = gpu_merge(gpu, n, periodic, x, pos, ndot, gpu.make_merge_params())
    assert len(got[1]) < members
    check_same(ref, got)


@pytest.mark.parametrize("n,r_max,dr", [(30, 8.0, 2.0), (31, 8.0, 2.0), (31, 14.5, 0.5),
                                        (31, 14.6, 7.3), (40, 14.5, 14.5), (40, 16.0, 4.0),
                                        (64, 0.5, 0.25)])
@pytest.mark.parametrize("periodic", [True, False])
def test_radius_reach(gpu, orc, n, r_max, dr, periodic):
    g = np.random.default_rng(n + int(10 * r_max))
    pos = W.uniform_positions(60, n, g)
    pos[:3] = [[0.5, 0.5, 0.5], [n - 0.5, 0.2, n / 2], [n - 0.1, n - 0.1, n - 0.1]]
    ndot = W.lognormal_values(60, 1e50, 2.0, g)
    x = np.full((n, n, n), 0.99)
    x[g.random((n, n, n)) < 0.05] = 0.0
    kw = dict(dr=dr, r_max=r_max, f_ov=0.2)
    ref = orc.merge_sources(orc.make_merge_params(**kw), n, periodic, x, pos, ndot)
    check_same(ref, gpu_merge(gpu, n, periodic, x, pos, ndot, gpu.make_merge_params(**kw)))
