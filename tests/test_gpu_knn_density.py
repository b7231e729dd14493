"""Neighbour sets of points of uneven density, where the search takes its first block of cells from the counts
around the query: the sets against the oracle, and the time against that of even density."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def v():
    import paper_2403_07412_amd as v
    v.library()
    return v


def _sites(kind, n, rng):
    x = rng.uniform(size=(n, 2))
    if kind == "outliers":  # all but a few points in a few of the cells
        x[rng.choice(n, 6, replace=False)] = rng.uniform(-9, 9, (6, 2))
    elif kind == "city":    # half of the points in a ten-thousandth of the area
        x[:n // 2] = 0.5 + 0.005 * rng.standard_normal((n // 2, 2))
    elif kind == "corner":  # the densest cells at the edge of the grid
        x[n // 10:] = 0.003 * np.abs(rng.standard_normal((n - n // 10, 2)))
    elif kind == "line":
        x[:, 1] = x[:, 0] + 1e-5 * rng.standard_normal(n)
    elif kind == "heap":    # many coincident points
        x[n // 2:] = x[rng.integers(0, 40, n - n // 2)]
    return np.ascontiguousarray(x[rng.permutation(n)])


@pytest.mark.parametrize("kind", ["outliers", "city", "corner", "line", "heap"])
@pytest.mark.parametrize("m", [1, 10, 64, 65, 150])
def test_sets_of_uneven_points(v, kind, m):
    import torch
    x = _sites(kind, 20_000, np.random.default_rng(8300 + m))
    rows = np.unique(np.concatenate([np.arange(8190, 8240), np.random.default_rng(m).integers(8192, len(x), 400)]))
    got = v.vecchia_knn(torch.from_numpy(x).cuda(), m).cpu().numpy()
    np.testing.assert_array_equal(got[rows], oracle.knn_rows(x, m, rows=rows))


@pytest.mark.parametrize("kind", ["outliers", "city"])
@pytest.mark.parametrize("metric", [0, 1])
def test_queries_among_uneven_points(v, kind, metric):
    import torch
    rng = np.random.default_rng(8400)
    x, q = _sites(kind, 20_000, rng), _sites(kind, 300, rng)
    got = v.vecchia_knn_query(torch.from_numpy(x).cuda(), torch.from_numpy(q).cuda(), 40, metric=metric).cpu().numpy()
    np.testing.assert_array_equal(got, oracle.knn_query(x, q, 40, metric))


def test_a_dense_place_does_not_multiply_the_work(v):
    """Half of 200,000 points in a small part of the area: a block sized for the average count reads thousands
    of points a query there (14 times the time of even points; sized from the counts, 3 times)."""
    import torch

    def best(x, m=60):
        t = torch.from_numpy(x).cuda()
        out = torch.empty((len(x), m), dtype=torch.int32, device="cuda")
        ws = torch.empty(v.vecchia_knn_workspace_size(len(x)), dtype=torch.uint8, device="cuda")
        times = []
        for _ in range(12):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            v.vecchia_knn(t, m, out=out, ws=ws)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
        return min(times)

    rng = np.random.default_rng(8500)
    even, uneven = _sites("even", 200_000, rng), _sites("city", 200_000, rng)
    assert best(uneven) < 7 * best(even)
