"""Reweighting of populations and pools too large for one workgroup: against the oracle around the size where the
launches change, with particles of no finite likelihood, and over several runs."""
import math

import numpy as np
import pytest
import torch

from paper_2601_02336_amd import synth
from paper_2601_02336_amd.synth import Bound
from oracle import oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def smcgw():
    from paper_2601_02336_amd import smcgw as m
    return m


def _check(b, b_ref, dz, dz_ref, anc, anc_ref):
    # beta is a point of the bisection's 1e-14 grid; the evidence is a sum of P terms in FP64
    assert abs(b - b_ref) <= 1e-12 * max(1.0, abs(b_ref)) + 2e-14
    assert abs(dz - dz_ref) <= 1e-9 * max(1.0, abs(dz_ref))
    assert np.mean(anc == anc_ref) >= 0.999


@pytest.mark.parametrize("P", [2560, 2561, 2624, 8193, 32768, 32769, 61440, 300000])
@pytest.mark.parametrize("alpha,beta_prev,scale", [(0.95, 0.0, 40.0), (0.5, 0.3, 40.0), (0.9, 0.2, 1e-3)])
def test_population(smcgw, P, alpha, beta_prev, scale):
    """scale 1e-3: nearly equal weights, beta jumps to 1."""
    rng = np.random.default_rng(P)
    D = 3
    logl = -0.5 * rng.chisquare(11, P) * scale - 3000.0
    logl[::97] = -np.inf
    logl[::101] = np.nan
    x, g = rng.normal(size=(P, D)), rng.normal(size=(P, D))
    carry = rng.integers(0, 1000, P).astype(np.int32)
    ll_ref = np.where(np.isnan(logl), -np.inf, logl)
    rc, b_ref, dz_ref, w_ref = O.smc_reweight(ll_ref, beta_prev, alpha)
    anc_ref = O.resample(w_ref, seed=77, iteration=3)
    c = smcgw.Context(0)
    xt, lt, gt, ct = (torch.tensor(a, device="cuda") for a in (x, logl, g, carry))
    b, dz, anc = c.smc_reweight_resample(xt, lt, gt, beta_prev, alpha, seed=77, iteration=3, carry=ct)
    c.close()
    a = anc.cpu().numpy()
    _check(b, b_ref, dz, dz_ref, a, anc_ref)
    assert np.all(np.isfinite(logl[a]))
    np.testing.assert_array_equal(xt.cpu().numpy(), x[a])
    np.testing.assert_array_equal(lt.cpu().numpy(), logl[a])
    np.testing.assert_array_equal(gt.cpu().numpy(), g[a])
    np.testing.assert_array_equal(ct.cpu().numpy(), carry[a])


def test_no_finite_likelihood(smcgw):
    """As for a small population: beta stays, the increment is -inf, the temperature cannot advance."""
    c = smcgw.Context(0)
    for P in (500, 9000):
        x = torch.arange(P, dtype=torch.float64, device="cuda")[:, None].contiguous()
        ll = torch.full((P,), -math.inf, dtype=torch.float64, device="cuda")
        out = torch.zeros(2, dtype=torch.float64, device="cuda")
        anc = c.smc_reweight_resample_async(x, ll, None, 0.25, 0.9, 1, 0, out)
        assert out[0].item() == 0.25 and out[1].item() == -math.inf
        assert torch.all(anc == P - 1)
        with pytest.raises(smcgw.SmcgwError):
            c.smc_reweight_resample(x, ll, None, 0.25, 0.9, 1, 0)
    c.close()


@pytest.mark.parametrize("T,N", [(5, 512), (13, 197), (30, 2048), (97, 700), (1, 9000)])
def test_pool(smcgw, T, N):
    """T = 97: a ladder too long for the kernel arguments."""
    rng = np.random.default_rng(T)
    betas = np.concatenate([[0.0], np.geomspace(1e-3, 0.3, T - 1)]) if T > 1 else np.zeros(1)
    var = 1.0 / (1.0 + 500.0 * betas)
    x = rng.standard_normal((T, N, 4)) * np.sqrt(var)[:, None, None]
    ll = (-250.0 * (x ** 2).sum(2)).reshape(T * N)
    logz = 2.0 * np.log(var)
    ll[::89] = -np.inf
    x = x.reshape(T * N, 4)
    rc, b_ref, lz_ref, w = O.ps_reweight(ll.reshape(T, N), betas.tolist(), logz.tolist(), betas[-1], 0.7)
    anc_ref = O.resample_n(w, N, 5, 2)
    c = smcgw.Context(0)
    xp, lp = torch.tensor(x, device="cuda"), torch.tensor(ll, device="cuda")
    gp = (2.0 * xp).contiguous()
    th, lt, gt = torch.empty((N, 4), dtype=torch.float64, device="cuda"), torch.empty(N, dtype=torch.float64, device="cuda"), \
        torch.empty((N, 4), dtype=torch.float64, device="cuda")
    b, lz, anc = c.ps_reweight_resample(xp, lp, gp, betas.tolist(), logz.tolist(), 0.7, 5, 2, th, lt, gt)
    a = anc.cpu().numpy()
    _check(b, b_ref, lz, lz_ref, a, anc_ref)
    np.testing.assert_array_equal(th.cpu().numpy(), x[a])
    np.testing.assert_array_equal(lt.cpu().numpy(), ll[a])
    np.testing.assert_array_equal(gt.cpu().numpy(), 2.0 * x[a])
    # the drawn population written over the pool's first rows: the same points
    b2, lz2, anc2 = c.ps_reweight_resample(xp, lp, gp, betas.tolist(), logz.tolist(), 0.7, 5, 2, xp[:N], lp[:N], gp[:N])
    assert b2 == b and lz2 == lz and torch.equal(anc2, anc)
    assert torch.equal(xp[:N], th) and torch.equal(lp[:N], lt) and torch.equal(gp[:N], gt)
    c.close()


def test_runs_in_one_call(smcgw):
    """Two runs of 8200 particles in one iteration call: each is bit for bit the run alone."""
    D, P = 3, 8200
    bounds = [Bound(-5.0, 5.0, synth.BND_REFLECT, synth.PRIOR_UNIFORM)] * D
    c = smcgw.Context(0)
    c.set_prior(bounds)
    c.set_target(synth.TARGET_GAUSS, D)
    x = torch.tensor(synth.prior_draw(np.random.default_rng(1), 2 * P, bounds), device="cuda")
    kw = dict(alpha=0.9, step=0.3, max_depth=3, shrink=0.0, precision=smcgw.PLAIN_FP64, history_cap=4)
    both = smcgw.SmcRuns(c, x, 2, seed=11, **kw)
    for _ in range(3):
        both.step()
    for r in range(2):
        one = smcgw.SmcRuns(c, x[r * P:(r + 1) * P].contiguous(), 1, seed=11 + r, **kw)
        for _ in range(3):
            one.step()
        assert torch.equal(both.theta[both.run_slice(r)], one.theta)
        assert np.array_equal(both.state()[r], one.state()[0]) and np.array_equal(both.history()[r], one.history()[0])
    c.close()
