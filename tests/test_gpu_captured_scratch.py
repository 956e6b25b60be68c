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


def test_iteration_graph(smcgw):
    """The graph of an iteration, and between its replays eager work on the same context that needs larger scratch: a
    larger population (the covariance's and the reweighting's) and a pool."""
    D = 3
    bounds = [synth.Bound(-5.0, 5.0, synth.BND_REFLECT, synth.PRIOR_UNIFORM)] * D
    kw = dict(alpha=0.9, step=0.3, max_depth=3, shrink=0.0, seed=5, precision=smcgw.PLAIN_FP64, history_cap=8)

    def context():
        c = smcgw.Context(0)
        c.set_prior(bounds)
        c.set_target(synth.TARGET_GAUSS, D)
        return c
    x = torch.tensor(synth.prior_draw(np.random.default_rng(1), 400, bounds), device="cuda")
    a, b = context(), context()
    graphed, eager = smcgw.SmcRuns(a, x, 2, **kw), smcgw.SmcRuns(b, x, 2, **kw)
    graph = graphed.graph()
    for n in (0, 60000, 300000, 300000):
        if n:
            big = smcgw.SmcRuns(a, torch.tensor(synth.prior_draw(np.random.default_rng(n), n, bounds), device="cuda"), 1, **kw)
            big.step()
            out = [torch.empty((1000, D), dtype=torch.float64, device="cuda"),
                   torch.empty(1000, dtype=torch.float64, device="cuda")]
            a.ps_reweight_resample(big.theta[:50000].contiguous(), big.logl[:50000].contiguous(), None, [0.1] * 50,
                                   [0.0] * 50, 0.5, 1, 1, *out, None)
        graph.launch()
        eager.step()
        torch.cuda.synchronize()
        assert torch.equal(graphed.theta, eager.theta) and torch.equal(graphed.logl, eager.logl)
        assert np.array_equal(graphed.state(), eager.state()) and np.array_equal(graphed.history(), eager.history())
    graph.close()
    a.close()
    b.close()


def test_sweeps_graph(smcgw):
    """The sweeps keep a graph of their own between calls: a larger batch of the plain form in between."""
    ev = event(synth.EventSpec(20.0, 20.0 + 999 * 0.5, 0.5, 2, 20.0, 83))
    b = synth.gw_prior_for(ev)
    c = smcgw.Context(0)
    c.add_event(ev)
    c.set_prior(b)
    c.set_target(synth.TARGET_GW, 11)
    x = torch.tensor(synth.prior_draw(np.random.default_rng(6), 3000, b), device="cuda")
    x0 = x[:40].contiguous()
    ll0, g0 = c.loglike_grad_tangent(x0)
    chol = torch.diag(torch.tensor([(q.hi - q.lo) * 0.01 for q in b], dtype=torch.float64, device="cuda"))
    y = [x0.clone(), ll0.clone(), g0.clone()]
    ref = None
    for n in (40, 600, 3000):
        c.loglike_grad_tangent(x[:n].contiguous())
        for dst, src in zip(y, (x0, ll0, g0)):
            dst.copy_(src)
        c.nuts_step_sweeps(*y, chol, step=0.2, beta=0.1, seed=1, iteration=1, max_depth=4)
        torch.cuda.synchronize()
        ref = ref or [t.clone() for t in y]
        assert all(torch.equal(u, v) for u, v in zip(y, ref))
    c.close()
