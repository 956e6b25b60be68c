"""Captured calls whose scratch is outgrown by later eager calls: the graph's replays still give the eager results."""
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


def _capture(call):
    graph = torch.cuda.CUDAGraph()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.graph(graph, stream=s):
        call()
    return graph


def test_start_order_of_a_batch(smcgw):
    """A batch over events of different lengths, captured with its start order in scratch; then two eager batches
    that need a larger one (the first holds 4096 particles)."""
    evs = [event(synth.EventSpec(20.0, 20.0 + (n - 1) * 0.5, 0.5, 2, 20.0, 70 + n)) for n in (700, 9000, 100)]
    rng = np.random.default_rng(3)
    x = torch.tensor(synth.prior_draw(rng, 9000, synth.gw_prior_for(evs[0])), device="cuda")
    of = torch.tensor(rng.integers(0, 3, 9000).astype(np.int32), device="cuda")
    c = smcgw.Context(0)
    for e in evs:
        c.add_event(e)
    P = 2000
    xs, ofs = x[:P].contiguous(), of[:P].contiguous()
    ref = c.loglike_grad(xs, event_of_particle=ofs)
    ll, g = torch.zeros(P, dtype=torch.float64, device="cuda"), torch.zeros_like(xs)
    graph = _capture(lambda: c.loglike_grad(xs, ll, g, event_of_particle=ofs))
    for n in (P, 5000, 9000):
        big = c.loglike_grad(x[:n].contiguous(), event_of_particle=of[:n].contiguous())
        assert torch.equal(big[0][:P], ref[0]) and torch.equal(big[1][:P], ref[1])
        for _ in range(2):
            ll.zero_()
            g.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(ll, ref[0]) and torch.equal(g, ref[1])
    c.close()


def test_segments_of_few_particles(smcgw):
    """A call of few particles on a long event, captured with its segments' scratch; then eager calls that need more."""
    ev = event(synth.EventSpec(20.0, 20.0 + 20000 * 0.5, 0.5, 2, 20.0, 81))
    x = torch.tensor(synth.prior_draw(np.random.default_rng(4), 600, synth.gw_prior_for(ev)), device="cuda")
    c = smcgw.Context(0)
    c.add_event(ev)
    for prec in (smcgw.MIXED, smcgw.PLAIN_FP64):
        xs = x[:5].contiguous()
        ref = c.loglike_grad(xs, precision=prec)
        ll, g = torch.zeros(5, dtype=torch.float64, device="cuda"), torch.zeros_like(xs)
        graph = _capture(lambda: c.loglike_grad(xs, ll, g, precision=prec))
        for n in (5, 90, 250, 600):
            big = c.loglike_grad(x[:n].contiguous(), precision=prec)
            assert torch.equal(big[0][:5], ref[0]) and torch.equal(big[1][:5], ref[1])
            for _ in range(2):
                ll.zero_()
                g.zero_()
                graph.replay()
                torch.cuda.synchronize()
                assert torch.equal(ll, ref[0]) and torch.equal(g, ref[1])
    c.close()
