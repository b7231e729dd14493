"""The rows kernel (four conditionals per wavefront; the one-wavefront variant up to four tile rows) at the
sizes where it can go wrong: full and nearly empty last tiles, the first points with their short sets, item
counts that do not fill a wavefront, wavefronts that mix set sizes, fields and parameter vectors, and a
failing conditional beside sound ones.  Tolerances are those of the variant tests (1e-10 on totals, 1e-9 on
terms)."""
import numpy as np
import pytest

import oracle
import workloads as wl
from util import assert_grad_close, assert_total_close, to_device

pytestmark = pytest.mark.gpu

# m + 2 rows: 16, 32, 48 and 64 fill 1 .. 4 tile rows
MS = [0, 1, 2, 13, 14, 15, 29, 30, 31, 45, 46, 47, 61, 62]


@pytest.fixture(scope="module")
def lib():
    import paper_2403_07412_amd as v
    v.library()
    return v


@pytest.mark.parametrize("m", MS)
def test_terms_from_the_first_point_on(lib, m):
    import torch
    rng = np.random.default_rng(7100 + m)
    f = wl.small_field(rng, 2 * m + 19, m, [0.5, 1.5, 2.5][m % 3], (1.3, 0.09, 4e-4))
    locs, z, nbr, theta = to_device(f)
    ell, gref = oracle.terms(f.locs, f.z, f.nbr, m, f.nu, f.thetas[0], with_grad=True)
    for grad in (False, True):
        t, g, st = lib.vecchia_loglik_terms_variant(locs, z, nbr, m, f.nu, theta, "tile_w1", with_grad=grad)
        torch.cuda.synchronize()
        assert int(st.item()) == 0
        np.testing.assert_allclose(t.cpu().numpy(), ell, rtol=1e-9, atol=1e-11)
        if grad:
            np.testing.assert_allclose(g.cpu().numpy(), gref, rtol=2e-7, atol=1e-9 * np.abs(gref).max())


@pytest.mark.parametrize("ntheta", [1, 3, 4])
@pytest.mark.parametrize("with_grad", [False, True])
def test_plan_mixing_fields_in_a_wavefront(lib, ntheta, with_grad):
    """Tiny fields of several set sizes share tile classes, so wavefronts span fields; every evaluation has
    the bits of its single call."""
    import torch
    rng = np.random.default_rng(7200 + ntheta)
    fields = [wl.small_field(rng, n, m, 1.5, (1.0, 0.1, 1e-3))
              for n, m in [(3, 5), (17, 9), (40, 14), (33, 16), (50, 22), (61, 30), (64, 31), (70, 40), (90, 46), (95, 55), (80, 62)]]
    dev = [to_device(f)[:3] for f in fields]
    th = np.stack([rng.uniform(0.5, 2.0, (len(fields), ntheta)), rng.uniform(0.02, 0.2, (len(fields), ntheta)),
                   rng.uniform(1e-4, 1e-3, (len(fields), ntheta))], axis=2)
    thetas = torch.from_numpy(th).cuda()
    plan = lib.BatchedPlan([(*d, f.m) for d, f in zip(dev, fields)], ntheta, 1.5, with_grad)
    out, grad, status = plan(thetas)
    torch.cuda.synchronize()
    assert int(status.abs().max().item()) == 0
    for a, (d, f) in enumerate(zip(dev, fields)):
        for q in range(ntheta):
            o, g, st = lib.vecchia_loglik_variant(*d, f.m, 1.5, thetas[a, q].contiguous(), "tile_w1",
                                                  with_grad=with_grad)
            torch.cuda.synchronize()
            assert int(st.item()) == 0
            assert o.item() == out[a, q].item(), (f.n, f.m, q)
            if with_grad:
                assert torch.equal(g, grad[a, q]), (f.n, f.m, q)
            ell, gref = oracle.terms(f.locs, f.z, f.nbr, f.m, 1.5, th[a, q], with_grad=True)
            assert_total_close(o.item(), oracle.compensated_sum(ell), 1e-10, f"n={f.n} m={f.m}")
            if with_grad:
                assert_grad_close(g.cpu().numpy(), [oracle.compensated_sum(gref[:, p]) for p in range(3)],
                                  np.abs(gref).sum(0), 1e-9, f"n={f.n} m={f.m}")


@pytest.mark.parametrize("m", [9, 25, 40, 57])
@pytest.mark.parametrize("kind", ["nan", "index", "singular"])
def test_failing_point_leaves_its_neighbours_alone(lib, m, kind):
    import torch
    rng = np.random.default_rng(7300 + m)
    f = wl.small_field(rng, 200, m, 0.5, (1.0, 0.2, 0.0))
    at = 150
    locs, z, nbr = f.locs.copy(), f.z.copy(), f.nbr.copy()
    if kind == "nan":
        z[at] = np.nan
        bad = [i for i in range(200) if i == at or at in nbr[i, :min(i, m)]]
    elif kind == "index":
        nbr[at, 0] = at  # not an earlier point
        bad = [at]
    else:
        nbr[at, 1] = nbr[at, 0]  # the same neighbour twice and no nugget
        bad = [at]
    ell, _ = oracle.terms(f.locs, f.z, f.nbr, m, 0.5, f.thetas[0], with_grad=True)
    d = [torch.from_numpy(a).cuda() for a in (locs, z, nbr)]
    theta = torch.from_numpy(f.thetas[0].copy()).cuda()
    for grad in (False, True):
        t, _, st = lib.vecchia_loglik_terms_variant(*d, m, 0.5, theta, "tile_w1", with_grad=grad)
        torch.cuda.synchronize()
        t = t.cpu().numpy()
        assert int(st.item()) == bad[0] + 1
        assert np.isnan(t[bad]).all()
        good = np.setdiff1d(np.arange(200), bad)
        np.testing.assert_allclose(t[good], ell[good], rtol=1e-9, atol=1e-11)


@pytest.mark.parametrize("m,nq", [(5, 1), (14, 30), (30, 33), (46, 65), (62, 7)])
def test_kriging(lib, m, nq):
    import torch
    rng = np.random.default_rng(7400 + m)
    xy, q, z = rng.uniform(0, 1, (120, 2)), rng.uniform(0, 1, (nq, 2)), rng.standard_normal(120)
    theta = np.array([1.1, 0.15, 1e-3])
    d = [torch.from_numpy(a).cuda() for a in (xy, z, q)]
    nbr = lib.vecchia_knn_query(d[0], d[2], m)
    lib.vecchia_set_variant(m, False, "tile_w1")
    try:
        mean, var, st = lib.vecchia_predict(d[0], d[1], d[2], nbr, m, (lib.MATERN, lib.EUCLIDEAN, 1.5),
                                            torch.from_numpy(theta).cuda())
        torch.cuda.synchronize()
    finally:
        lib.vecchia_set_variant(m, False, "auto")
    assert int(st.item()) == 0
    sets = nbr.cpu().numpy()
    for t in range(nq):
        p = np.vstack([xy[sets[t]], q[t:t + 1]])
        r = np.sqrt(((p[:, None] - p[None]) ** 2).sum(-1)) / theta[1]
        c = theta[0] * (1 + r) * np.exp(-r) + theta[2] * np.eye(m + 1)
        w = np.linalg.solve(c[:m, :m], c[:m, m])
        assert abs(mean[t].item() - w @ z[sets[t]]) <= 1e-9 * max(1.0, np.abs(w).sum())
        assert abs(var[t].item() - (c[m, m] - w @ c[:m, m])) <= 1e-9
