"""Ranges so short that the exponential leaves the double range: e^-r must take the powers of r that multiply
it to zero with it, in the covariance and in its beta-derivative."""
import mpmath
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

CODES = [(0, 0, 0.5), (0, 0, 1.5), (0, 0, 2.5), (1, 0, 0.9), (0, 1, 1.5), (0, 1, 2.5), (1, 1, 0.9)]


@pytest.fixture(scope="module")
def v():
    import paper_2403_07412_amd as v
    v.library()
    return v


def _device(*arrays):
    import torch
    return [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in arrays]


@pytest.mark.parametrize("cov", CODES)
@pytest.mark.parametrize("m", [46, 62, 70, 90, 125, 150])  # derivative over the pairs, or kept by the tiled kernel
def test_uncorrelated_points(v, cov, m):
    uncorrelated_points(v, cov, m)


@pytest.mark.parametrize("cov", CODES)
@pytest.mark.parametrize("m", [1, 5, 14, 15, 30])
def test_uncorrelated_points_in_small_sets(v, cov, m):
    """Up to two tile rows the derivative stays in registers from the fill, the diagonal's included."""
    uncorrelated_points(v, cov, m)


def uncorrelated_points(v, cov, m):
    """Lattice points at least 0.5 apart under beta from 1e-60 down: every covariance is 0, so the terms are
    those of independent points and the beta-derivative is exactly 0."""
    import torch
    rng = np.random.default_rng(9100 + m)
    n = m + 9
    g = int(np.ceil(np.sqrt(n)))
    locs = 0.5 * np.stack(np.meshgrid(np.arange(g), np.arange(g)), -1).reshape(-1, 2)[:n] + [10.0, 20.0]
    z = rng.standard_normal(n)
    nbr = np.array([[j if j < min(i, m) else -1 for j in range(m)] for i in range(n)], dtype=np.int32)
    d = _device(locs, z, nbr)
    s2, t2 = 1.0, 0.1
    c = s2 + t2
    want = -0.5 * (np.log(2 * np.pi) + np.log(c) + z * z / c)
    gwant = 0.5 * (z * z / c - 1.0) / c
    for beta in (1e-60, 1e-78, 1e-80, 1e-104, 1e-140, 1e-155, 1e-200):
        theta = torch.tensor([s2, beta, t2], dtype=torch.float64, device="cuda")
        t, gr, st = v.vecchia_loglik_terms_cov(*d, m, cov, theta, with_grad=True)
        t0, _, st0 = v.vecchia_loglik_terms_cov(*d, m, cov, theta)
        torch.cuda.synchronize()
        assert int(st.item()) == 0 and int(st0.item()) == 0, beta
        for got in (t, t0):
            np.testing.assert_allclose(got.cpu().numpy(), want, rtol=0, atol=1e-14 * (1 + np.abs(want).max()))
        gr = gr.cpu().numpy()
        assert (gr[:, 1] == 0.0).all(), (beta, np.abs(gr[:, 1]).max())
        for p in (0, 2):
            np.testing.assert_allclose(gr[:, p], gwant, rtol=0, atol=1e-13 * (1 + np.abs(gwant).max()))


@pytest.mark.parametrize("nu", [0.5, 1.5, 2.5])
@pytest.mark.parametrize("variant", ["unblocked", "tile_w1"])
def test_two_points_at_the_end_of_the_range(v, nu, variant):
    """Two points 0.5 apart, r from 690 to 760: the covariance c is below 1e-295, so the derivative of the second
    term is z1 z2 / (s2 + t2)^2 dC/dbeta, here to 50 digits.  e^-r carries an absolute error of one denormal
    besides a relative one of a few roundings, both times r^p / beta."""
    import torch
    mpmath.mp.dps = 50
    locs, z = np.array([[0.0, 0.0], [0.5, 0.0]]), np.array([1.3, -0.7])
    nbr = np.array([[-1], [0]], dtype=np.int32)
    d = _device(locs, z, nbr)
    for r in (690.0, 707.0, 709.5, 720.0, 733.0, 744.0, 747.0, 760.0):
        beta = 0.5 / r
        theta = torch.tensor([1.0, beta, 0.1], dtype=torch.float64, device="cuda")
        _, g, st = v.vecchia_loglik_terms_variant(*d, 1, nu, theta, variant, with_grad=True)
        torch.cuda.synchronize()
        assert int(st.item()) == 0
        q = mpmath.mpf(0.5) / mpmath.mpf(beta)
        h = {0.5: q, 1.5: q ** 2, 2.5: q ** 2 * (1 + q) / 3}[nu]
        factor = mpmath.mpf(1.3) * mpmath.mpf(-0.7) / mpmath.mpf(1.1) ** 2 / mpmath.mpf(beta)
        want = h * mpmath.exp(-q) * factor
        tol = abs(want) * mpmath.mpf(1e-12) + abs(h * factor) * mpmath.mpf(5e-324)
        assert abs(mpmath.mpf(g[1, 1].item()) - want) <= tol, (r, g[1, 1].item(), float(want))
