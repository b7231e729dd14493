"""The built-in choice of kernel per tile rows and covariance code, at both ends of the tile classes where it
changes: totals and gradients against the oracle (1e-10, 1e-9 as everywhere), and for the Matern codes on
Euclidean distances the same bits with and without the gradient, in a plan and from the call without a
workspace."""
import numpy as np
import pytest

import oracle
import workloads as wl
from util import assert_grad_close, assert_total_close, to_device

pytestmark = pytest.mark.gpu

# m + 2 rows: 65 .. 80 are five tile rows, 81 .. 96 six, and so on to 162 (eleven)
ENDS = [62, 63, 78, 79, 94, 95, 110, 111, 126, 127, 142, 143, 158, 159, 160]


@pytest.fixture(scope="module")
def lib():
    import paper_2403_07412_amd as v
    v.library()
    return v


@pytest.mark.parametrize("m", ENDS)
def test_matern_forms_agree(lib, m):
    import torch
    nu = [0.5, 1.5, 2.5][m % 3]
    f = wl.small_field(np.random.default_rng(7700 + m), m + 60, m, nu, (1.1, 0.08, 1e-3))
    locs, z, nbr, theta = to_device(f)
    val, st0 = lib.vecchia_loglik(locs, z, nbr, m, nu, theta)
    out, grad, st1 = lib.vecchia_loglik_grad(locs, z, nbr, m, nu, theta)
    nout, ngrad, st2 = torch.empty_like(out), torch.empty_like(grad), torch.empty_like(st1)
    lib.vecchia_loglik_grad_noalloc(locs, z, nbr, m, nu, theta, nout, ngrad, st2)
    pv, _, _ = lib.BatchedPlan([(locs, z, nbr, m)], 1, nu, False)(theta.reshape(1, 1, 3).contiguous())
    pout, pgrad, _ = lib.BatchedPlan([(locs, z, nbr, m)], 1, nu, True)(theta.reshape(1, 1, 3).contiguous())
    torch.cuda.synchronize()
    assert [int(s.item()) for s in (st0, st1, st2)] == [0, 0, 0]
    assert {val.item(), out.item(), nout.item(), pv.item(), pout.item()} == {out.item()}
    assert torch.equal(grad, ngrad) and torch.equal(grad, pgrad.reshape(3))
    ell, gref = oracle.terms(f.locs, f.z, f.nbr, m, nu, f.thetas[0], with_grad=True)
    assert_total_close(out.item(), oracle.compensated_sum(ell), 1e-10, f"m={m}")
    assert_grad_close(grad.cpu().numpy(), [oracle.compensated_sum(gref[:, p]) for p in range(3)],
                      np.abs(gref).sum(0), 1e-9, f"m={m}")


@pytest.mark.parametrize("cov", [(1, 0, 0.9), (0, 1, 1.5), (1, 1, 0.9)])
@pytest.mark.parametrize("m", [46, 47, 62, 63, 78, 79, 142, 143, 158])
def test_other_codes_match_oracle(lib, cov, m):
    import torch
    rng = np.random.default_rng(7800 + m)
    n = m + 60
    locs = rng.uniform(size=(n, 2))
    theta = (1.1, 0.08, 1e-3)
    if cov[1]:
        locs = np.column_stack([-95 + 10 * locs[:, 0], 30 + 10 * locs[:, 1]])
        theta = (1.1, 60.0, 1e-2)
    z = rng.standard_normal(n)
    nbr = oracle.knn_rows(locs, m, metric=cov[1])
    dev = [torch.from_numpy(a).cuda() for a in (locs, z, nbr)]
    th = torch.tensor(theta, dtype=torch.float64, device="cuda")
    val, _, st0 = lib.vecchia_loglik_cov(*dev, m, cov, th)
    out, grad, st1 = lib.vecchia_loglik_cov(*dev, m, cov, th, with_grad=True)
    torch.cuda.synchronize()
    assert int(st0.item()) == 0 and int(st1.item()) == 0
    ell, gref = oracle.terms_cov(locs, z, nbr, m, cov, theta, with_grad=True)
    for got in (val, out):
        assert_total_close(got.item(), oracle.compensated_sum(ell), 1e-10, f"m={m}")
    assert_grad_close(grad.cpu().numpy(), [oracle.compensated_sum(gref[:, p]) for p in range(3)],
                      np.abs(gref).sum(0), 1e-9, f"m={m}")


@pytest.mark.parametrize("cov", [(1, 0, 0.9), (0, 1, 0.5), (0, 1, 1.5), (0, 1, 2.5), (1, 1, 0.9)])
@pytest.mark.parametrize("m", [159, 160])
def test_other_codes_with_eleven_tile_rows(lib, cov, m):
    test_other_codes_match_oracle(lib, cov, m)
