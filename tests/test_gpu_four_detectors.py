"""Four detectors, the most an event may have, through every form of the likelihood and of the transition: against the
oracle, and bit for bit the same in every batch, with and without the gradient, and at every slot width."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2601_02336_amd import synth
from oracle import oracle as O

from helpers import TOL, grad_err, logl_rel_err, widths

pytestmark = pytest.mark.gpu

OUT = ("n_leapfrog", "depth", "divergent", "accept_stat")


@pytest.fixture(scope="module")
def smc():
    from paper_2601_02336_amd import smcgw
    return smcgw


def _event(n, seed, df=0.5):
    """Three of the synthetic sites and a fourth, with an injection and noise as the others have."""
    sites = synth.synthetic_sites(3) + [synth.Site(-0.55, 2.0, 0.3, 0.3 + np.pi / 2)]
    rng = np.random.default_rng(seed)
    psd = np.stack([synth.power_law_psd(synth.freq_grid(20.0, df, n)) * s for s in (1.0, 1.0, 2.0, 1.5)])
    th = synth.prior_draw(rng, 1, synth.gw_bounds(300.0, 3000.0))[0]
    ev = synth.Event(20.0, df, n, sites, np.zeros((4, n), complex), psd, th, 0.0)
    th[4] *= np.sqrt(-2.0 * O.loglike_zero_data(ev, th)) / 20.0
    ev = dataclasses.replace(ev, theta_inj=th, snr_opt=20.0)
    return ev.with_data(O.waveform(ev, th) + synth.gaussian_noise(rng, psd, df))


# 310: one block; 3000, 4600: the grid on one wavefront and on a workgroup; 9000, 20000: several segments, 16 blocks
# each; 33500: 32 blocks each
@pytest.mark.parametrize("n", [310, 3000, 4600, 9000, 20000, 33500])
def test_likelihood(smc, n):
    ev = _event(n, n)
    b = synth.gw_prior_for(ev)
    x = torch.tensor(synth.prior_draw(np.random.default_rng(1), 2100, b), device="cuda")
    c = smc.Context(0)
    c.add_event(ev)
    pick = np.array([0, 1, 5, 2099])
    ll_ref, g_ref = O.loglike_grad(O.gw_target(ev), x[pick].cpu().numpy())
    for name, prec in (("mixed", smc.MIXED), ("plain", smc.PLAIN_FP64)):
        ll, g = c.loglike_grad(x, precision=prec)
        assert logl_rel_err(ll[pick].cpu().numpy(), ll_ref) <= TOL[name]["logl"]
        assert grad_err(g[pick].cpu().numpy(), g_ref, widths(b)) <= TOL[name]["grad"]
        for P in (1, 5, 31, 85, 250, 512, 700):
            a, d = c.loglike_grad(x[:P].contiguous(), precision=prec)
            assert torch.equal(a, ll[:P]) and torch.equal(d, g[:P]), (name, P)
            assert torch.equal(c.loglike_grad(x[:P].contiguous(), want_grad=False, precision=prec), ll[:P]), (name, P)
    c.close()


@pytest.mark.parametrize("n", [129, 513])
def test_last_block(smc, n):
    ev = _event(n, n)
    b = synth.gw_prior_for(ev)
    x = synth.prior_draw(np.random.default_rng(n), 9, b)
    ll_ref, g_ref = O.loglike_grad(O.gw_target(ev), x)
    c = smc.Context(0)
    c.add_event(ev)
    for name, prec in (("plain", smc.PLAIN_FP64), ("mixed", smc.MIXED)):
        ll, g = c.loglike_grad(torch.tensor(x, device="cuda"), precision=prec)
        assert logl_rel_err(ll.cpu().numpy(), ll_ref) <= TOL[name]["logl"]
        assert grad_err(g.cpu().numpy(), g_ref, widths(b)) <= TOL[name]["grad"]
    c.close()


# (bins, particles, precision): packed on one and on two blocks, two wavefronts, one particle per workgroup
@pytest.mark.parametrize("n,P,prec", [(310, 1281, 1), (310, 1281, 0), (900, 2561, 1), (900, 1537, 0), (900, 1300, 1)])
def test_transitions(smc, n, P, prec):
    ev = _event(n, n, df=2.0)
    b = synth.gw_prior_for(ev)
    c = smc.Context(0)
    c.add_event(ev)
    c.set_prior(b)
    c.set_target(synth.TARGET_GW, 11)
    x = torch.tensor(synth.prior_draw(np.random.default_rng(2), P, b), device="cuda")
    ll, g = c.loglike_grad(x, precision=prec)
    _, _, L = O.mass_matrix(x.cpu().numpy(), 0.0)
    chol = torch.tensor(L * 0.05, device="cuda")

    def step():
        y = [x.clone(), ll.clone(), g.clone()]
        o = c.nuts_step(*y, chol, step=0.2, beta=0.1, seed=7, iteration=3, max_depth=5, precision=prec)
        torch.cuda.synchronize()
        return y + [o[k] for k in OUT]
    first = step()
    assert int(first[4].max()) >= 4
    for width in (2, 4, 8):
        c.set_option(smc.OPT_NUTS_WAVES, width)
        assert all(torch.equal(u, v) for u, v in zip(first, step())), width
    # the log-likelihood and gradient that the transition left are those of its points
    name = "mixed" if prec == smc.MIXED else "plain"
    pick = np.arange(0, P, 400)
    ll_ref, g_ref = O.loglike_grad(O.gw_target(ev), first[0][pick].cpu().numpy())
    assert logl_rel_err(first[1][pick].cpu().numpy(), ll_ref) <= TOL[name]["logl"]
    assert grad_err(first[2][pick].cpu().numpy(), g_ref, widths(b)) <= TOL[name]["grad"]
    c.close()
