"""The local metric's four particles to a wavefront: remainders and mixed events."""
import numpy as np
import pytest
import torch

from paper_2601_02336_amd import synth

from helpers import event

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def smcgw():
    from paper_2601_02336_amd import smcgw as m
    return m


def _ctx(smcgw, ev, idx, b, events):
    c = smcgw.Context(0)
    for e in events:
        c.add_event(e)
    c.set_param_map(idx, ev.theta_inj)
    c.set_prior(b)
    c.set_target(synth.TARGET_GW, len(idx))
    return c


@pytest.mark.parametrize("n_par", [1, 4, 11])
def test_local_metric_remainders(smcgw, n_par):
    """A particle's factor, Fisher matrix and status do not depend on the particles that share its wavefront:
    counts around a multiple of four, two events in turn and a Fisher matrix that overflows among them (the
    fallback), each bit for bit against calls of one particle."""
    evs = [event(s) for s in synth.ragged_specs()[:4:2]]
    full = synth.gw_prior_for(evs[0])
    idx = [4, 0, 10, 1, 2, 3, 5, 6, 7, 8, 9][:n_par]
    b = [full[i] for i in idx]
    c = _ctx(smcgw, evs[0], idx, b, events=evs)
    x = synth.prior_draw(np.random.default_rng(43), 67, b)
    x[5, 0] = 1e-300   # luminosity distance
    fb = torch.tensor(np.tril(np.random.default_rng(44).normal(size=(n_par, n_par))), device="cuda")
    em = torch.tensor((np.arange(67) // 3 % 2).astype(np.int32), device="cuda")
    one = []
    for p in range(67):
        c.set_event_map(em[p:p + 1].contiguous())
        one.append(c.local_metric(torch.tensor(x[p:p + 1], device="cuda"), 0.3, fallback=fb, fisher=True))
    assert int(one[5][2][0]) == 1 and sum(int(o[2][0]) for o in one) == 1
    for P in (1, 3, 4, 5, 7, 8, 67):
        c.set_event_map(em[:P].contiguous())
        got = c.local_metric(torch.tensor(x[:P], device="cuda"), 0.3, fallback=fb, fisher=True)
        torch.cuda.synchronize()
        for k in range(3):
            want = torch.cat([o[k] for o in one[:P]])
            assert torch.equal(torch.nan_to_num(got[k].double()), torch.nan_to_num(want.double())), (P, k)
    c.close()
