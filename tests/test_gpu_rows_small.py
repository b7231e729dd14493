"""Launches of the rows kernel too small to fill the GPU give every conditional a wavefront, whose row groups
share its evaluations: the bits of the launches that hold four conditionals to a wavefront, at the ends of the
tile classes and of the sets' lengths, and less time than they."""
import numpy as np
import pytest

import workloads as wl
from util import to_device

pytestmark = pytest.mark.gpu

MATERN = [15, 16, 30, 31, 46, 47, 62]  # 17 .. 64 rows; one tile row keeps four to a wavefront
OTHER = [1, 2, 14, 15, 30]
CASES = [((0, 0, nu), m) for m in MATERN for nu in (0.5, 1.5, 2.5)] + \
        [(cov, m) for m in OTHER for cov in ((1, 0, 0.9), (0, 1, 0.5), (0, 1, 1.5), (0, 1, 2.5), (1, 1, 1.3))]


@pytest.fixture(scope="module")
def lib():
    import paper_2403_07412_amd as v
    v.library()
    return v


def _field(lib, cov, m, n):
    import torch
    rng = np.random.default_rng(9300 + m)
    locs = rng.uniform(size=(n, 2))
    theta = [1.2, 0.06, 1e-3]
    if cov[1]:
        locs = np.column_stack([-95 + 10 * locs[:, 0], 30 + 10 * locs[:, 1]])
        theta = [1.2, 50.0, 1e-2]
    locs, z = torch.from_numpy(np.ascontiguousarray(locs)).cuda(), torch.from_numpy(rng.standard_normal(n)).cuda()
    return locs, z, lib.vecchia_knn(locs, m, metric=cov[1]), torch.tensor(theta, dtype=torch.float64, device="cuda")


@pytest.mark.parametrize("cov,m", CASES)
def test_same_bits_as_four_to_a_wavefront(lib, cov, m):
    import torch
    locs, z, nbr, theta = _field(lib, cov, m, 3400)
    for grad in (False, True):
        t, g, st = lib.vecchia_loglik_terms_cov(locs, z, nbr, m, cov, theta, with_grad=grad)
        for n in (1, 2, 3, m, m + 1, m + 2, 1023, 1024, 1025):  # the first n points, as a field of their own
            ts, gs, ss = lib.vecchia_loglik_terms_cov(locs[:n].contiguous(), z[:n].contiguous(), nbr[:n].contiguous(),
                                                      m, cov, theta, with_grad=grad)
            torch.cuda.synchronize()
            assert int(st.item()) == 0 and int(ss.item()) == 0
            assert torch.equal(ts, t[:n]), n
            if grad:
                assert torch.equal(gs, g[:n]), n


@pytest.mark.parametrize("m", [25, 40, 57])
@pytest.mark.parametrize("ntheta", [1, 3, 4, 8])
def test_small_plans(lib, m, ntheta):
    """A plan of few items, vectors in groups of four among them, one invalid, against one of many."""
    import torch
    rng = np.random.default_rng(9400 + m)
    f = wl.small_field(rng, 90, m, 1.5, (1.0, 0.1, 1e-3))
    d = to_device(f)[:3]
    th = np.stack([rng.uniform(0.5, 2.0, (1, ntheta)), rng.uniform(0.02, 0.2, (1, ntheta)),
                   rng.uniform(1e-4, 1e-3, (1, ntheta))], axis=2)
    if ntheta > 1:
        th[0, 1, 0] = -1.0
    many = 60  # fields, 5,400 items and more
    few = lib.BatchedPlan([(*d, m)], ntheta, 1.5, True)(torch.from_numpy(th).cuda())
    all_ = lib.BatchedPlan([(*d, m)] * many, ntheta, 1.5, True)(torch.from_numpy(np.repeat(th, many, 0)).cuda())
    torch.cuda.synchronize()
    for a, b in zip(few, all_):
        assert torch.equal(a[0].cpu().nan_to_num(7.0), b[0].cpu().nan_to_num(7.0))
        assert torch.equal(b[0].cpu().nan_to_num(7.0), b[-1].cpu().nan_to_num(7.0))


@pytest.mark.parametrize("cov,m", [((0, 0, 1.5), 60), ((0, 1, 1.5), 30)])
def test_small_launch_does_not_wait_for_one_wavefront(lib, cov, m):
    """300 points against 4,000, which four to a wavefront take as long as (0.87 and 1.07 of their time)."""
    import torch

    def time(n):
        locs, z, nbr, theta = _field(lib, cov, m, n)
        ws = torch.empty(lib.vecchia_workspace_size(n, m), dtype=torch.uint8, device="cuda")
        lib.vecchia_loglik_cov(locs, z, nbr, m, cov, theta, with_grad=True, ws=ws)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for _ in range(20):
                lib.vecchia_loglik_cov(locs, z, nbr, m, cov, theta, with_grad=True, ws=ws)
        best = np.inf
        for _ in range(40):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            graph.replay()
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        return best

    assert time(300) < 0.78 * time(4000)
