"""Batches over events of very different lengths, whose particles start in an order of their own: around the size from
which they do, and around a workgroup's share of the ordering.  Every particle gets, bit for bit, what its event alone
gives."""
import numpy as np
import pytest
import torch

from paper_2601_02336_amd import synth

from helpers import event

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P", [1280, 1281, 4096, 4097, 16384, 40001])
@pytest.mark.parametrize("form", ["random", "rising", "one event"])
def test_start_order(P, form):
    from paper_2601_02336_amd import smcgw as smc
    evs = [event(synth.EventSpec(20.0, 20.0 + (n - 1) * 0.5, 0.5, 1, 20.0, 90 + n)) for n in (100, 8200, 1500, 700, 90)]
    rng = np.random.default_rng(P)
    of = rng.integers(-1, 7, P).astype(np.int32) if form == "random" else \
        np.sort(rng.integers(0, 5, P)).astype(np.int32) if form == "rising" else np.full(P, 3, np.int32)
    x = torch.tensor(synth.prior_draw(rng, P, synth.gw_prior_for(evs[0])), device="cuda")
    c = smc.Context(0)
    for e in evs:
        c.add_event(e)
    ll, g = torch.full((P,), float("nan"), dtype=torch.float64, device="cuda"), torch.full_like(x, float("nan"))
    c.timing(smc.KERNEL_PREP)
    c.loglike_grad(x, ll, g, event_of_particle=torch.tensor(of, device="cuda"))
    assert (c.timing_read(smc.KERNEL_PREP)[1] > 0) == (P > 1280)
    c.timing()
    for k, e in enumerate(evs):
        rows = torch.tensor(np.nonzero(np.clip(of, 0, 4) == k)[0], device="cuda")
        one = smc.Context(0)
        one.add_event(e)
        a, b = one.loglike_grad(x[rows].contiguous())
        assert torch.equal(a, ll[rows]) and torch.equal(b, g[rows])
        one.close()
    c.close()


def test_near_lengths_keep_index_order():
    """Lengths within a factor of two, and short events: no order is made."""
    from paper_2601_02336_amd import smcgw as smc
    for ns in ((8000, 8200), (300, 600, 4000)):
        evs = [event(synth.EventSpec(20.0, 20.0 + (n - 1) * 0.5, 0.5, 1, 20.0, 90 + n)) for n in ns]
        x = torch.tensor(synth.prior_draw(np.random.default_rng(1), 3000, synth.gw_prior_for(evs[0])), device="cuda")
        c = smc.Context(0)
        for e in evs:
            c.add_event(e)
        c.timing(smc.KERNEL_PREP)
        c.loglike_grad(x, event_of_particle=torch.tensor((np.arange(3000) % len(ns)).astype(np.int32), device="cuda"))
        assert c.timing_read(smc.KERNEL_PREP)[1] == 0
        c.close()
