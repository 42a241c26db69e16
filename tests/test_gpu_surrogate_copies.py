"""The surrogate's BF16 weight copies follow its parameters through captured
graphs."""
import pytest
import torch

import paper_1709_09763_amd as P
from tests import inputs
from tests.gpu_util import case, device, host, to_dev

pytestmark = pytest.mark.gpu

K, M = 12, 3


def _ctx(hidden=64, l=3):
    c = P.Context(l, l, K, 1.0, 0.3, M, 0.01)
    P.mls2mc_surrogate_init(c.h, hidden, 1024, 3)
    return c


def _network(c, seed):
    n = P.mls2mc_surrogate_n_params(c.h)
    return to_dev(0.3 * inputs.rng(seed).standard_normal(n), torch.float32)


def _predict(c, x):
    G = torch.empty((x.shape[0], M * M), dtype=torch.float64, device="cuda:0")
    P.mls2mc_surrogate_predict(c.h, x, G)
    return G


def _captured(f):
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        f()  # sizes every workspace
    torch.cuda.current_stream().wait_stream(side)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        f()
    return g


def test_replayed_prediction_uses_the_parameters_set_since():
    device()
    case("captured surrogate_predict, parameters set before each replay")
    c, ref = _ctx(), _ctx()
    x = to_dev(inputs.theta_batch(1, 70, K))
    P.mls2mc_surrogate_set_params(c.h, _network(c, 0))
    G = torch.empty((70, M * M), dtype=torch.float64, device="cuda:0")
    g = _captured(lambda: P.mls2mc_surrogate_predict(c.h, x, G))
    for seed in (1, 2, 3):
        p = _network(c, seed)
        P.mls2mc_surrogate_set_params(c.h, p)
        P.mls2mc_surrogate_set_params(ref.h, p)
        g.replay()
        want = _predict(ref, x)
        torch.cuda.synchronize()
        assert torch.equal(G, want), seed
        assert torch.equal(_predict(c, x), want), seed


def test_eager_calls_after_a_capture_use_the_current_parameters():
    device()
    case("parameters set, predict captured, eager calls before the first replay")
    c, ref = _ctx(), _ctx()
    x = to_dev(inputs.theta_batch(2, 33, K))
    th, t = to_dev(inputs.theta_batch(3, 64, K)), to_dev(inputs.theta_batch(4, 64, M * M))
    for q in (c, ref):  # a capture also fixes whether inputs are standardised: train before it
        P.mls2mc_surrogate_add_pairs(q.h, th, t)
        P.mls2mc_surrogate_train(q.h, 1, 32, 1e-2, 0)
    p = _network(c, 5)
    P.mls2mc_surrogate_set_params(c.h, p)
    P.mls2mc_surrogate_set_params(ref.h, p)
    G = torch.empty((33, M * M), dtype=torch.float64, device="cuda:0")
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        P.mls2mc_surrogate_predict(c.h, x, G)
    want = _predict(ref, x)
    assert torch.equal(_predict(c, x), want)
    for q in (c, ref):
        P.mls2mc_surrogate_train(q.h, 1, 32, 1e-2, 1)
    want = _predict(ref, x)
    assert torch.equal(_predict(c, x), want)
    for _ in range(2):
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(G, want)


def test_replayed_delayed_acceptance_uses_the_parameters_set_since():
    device()
    case("captured pcn_step_da, parameters set before each replay")
    N, l = 130, 3
    c, ref = _ctx(l=l), _ctx(l=l)
    th0 = to_dev(inputs.theta_batch(6, N, K))
    G0 = c.forward(l, th0)
    y = G0[0].clone()
    phi0 = c.loglik(G0, y)
    xi = to_dev(inputs.theta_batch(7, N, K))
    u1, u2 = to_dev(1.0 - inputs.uniforms53(8, N)), to_dev(1.0 - inputs.uniforms53(9, N))

    def state():
        return [th0.clone(), G0.clone(), phi0.clone(), torch.empty(N, dtype=torch.uint8, device="cuda:0"),
                torch.empty(N, dtype=torch.uint8, device="cuda:0")]

    def step(q, s):
        P.mls2mc_pcn_step_da(q.h, l, l, 0.01, 1.0, 0.5, s[0], s[1], None, s[2], None, y, xi, u1, u2, s[3], s[4])

    P.mls2mc_surrogate_set_params(c.h, _network(c, 10))
    s = state()
    g = _captured(lambda: step(c, s))
    screened = set()
    for seed in (11, 12):
        p = _network(c, seed)
        P.mls2mc_surrogate_set_params(c.h, p)
        P.mls2mc_surrogate_set_params(ref.h, p)
        for a, b in zip(s, (th0, G0, phi0)):
            a.copy_(b)
        g.replay()
        r = state()
        step(ref, r)
        torch.cuda.synchronize()
        for a, b in zip(s, r):
            assert torch.equal(a, b), seed
        screened.add(host(r[4]).tobytes())
    assert len(screened) == 2  # the networks differ in what they let through
