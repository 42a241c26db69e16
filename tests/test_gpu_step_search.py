"""The adaptive step between 2049 and 4096 particles, which brackets the root
before it bisects, against the oracle's plain bisection."""
import numpy as np
import pytest

import oracle
import paper_1709_09763_amd as P
from tests import inputs
from tests.gpu_util import case, device, host, rel_err, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    device()
    c = P.Context(3, 3, 4, 1.0, 0.3, 2, 0.01)
    yield c
    c.close()


def _distances(kind, N, g):
    if kind == "wide":  # a first tempering step: the root next to the smallest step
        return 2e5 * g.chisquare(9, N)
    if kind == "narrow":  # the root next to the right end
        d = g.standard_normal(N)
        return d * (0.84 / d.std())
    if kind == "heavy":
        return np.exp(3.0 * g.standard_normal(N))
    if kind == "shifted":  # a large common part
        return 1e6 + 30.0 * g.standard_normal(N)
    d = np.zeros(N)  # "two": two values
    d[: N // 4] = 3.0
    return g.permutation(d) + 1e-3 * g.standard_normal(N)


@pytest.mark.parametrize("N", [2048, 2049, 4096, 4097, 8191, 8192, 8193])
@pytest.mark.parametrize("kind", ["wide", "narrow", "heavy", "shifted", "two"])
@pytest.mark.parametrize("tau", [0.5, 0.8])
def test_step_search(ctx, N, kind, tau):
    """The sums' relative error, about N^(1/2) 2^-53, moves the root by that over
    the slope of log ESS in log t, here above 0.05 ("shifted": the distances
    themselves carry 1e6 2^-53 / 30 = 4e-12): 1e-12, 1e-10 there, of t."""
    case(f"next_step search N={N} {kind} tau={tau}")
    d = _distances(kind, N, inputs.rng(N + len(kind)))
    out3, logw, w = ctx.next_step(to_dev(d), 1.0, 0.0, tau * N, 1e-6)
    o, ref = host(out3), oracle.next_step(d, 1.0, 0.0, tau * N, 1e-6)
    tol = 1e-10 if kind == "shifted" else 1e-12
    assert abs(o[0] - ref["next"]) <= tol * ref["next"]
    assert abs(o[1] - ref["dlogZ"]) <= 10 * tol * max(1.0, abs(ref["dlogZ"]))
    assert abs(o[2] - ref["ess"]) <= 10 * tol * N
    assert rel_err(host(w), ref["w"]) <= 100 * tol
    # the step is the last one at which ESS reaches the target
    if o[0] < 1.0 and o[0] > 1e-6:
        assert o[2] >= tau * N


@pytest.mark.parametrize("N", [2049, 5000])
def test_step_search_without_a_root(ctx, N):
    """Equal distances (ESS = N throughout), differences that overflow the weights,
    targets no ESS reaches, non-finite distances."""
    case(f"next_step search N={N} degenerate")
    o = host(ctx.next_step(to_dev(np.full(N, 7.0)), 1.0, 0.3, 0.5 * N)[0])
    assert o[0] == 1.0 and abs(o[2] - N) < 1e-9 * N
    d = np.where(np.arange(N) % 2 == 0, 0.0, 1e308)
    ref = oracle.next_step(d, 1.0, 0.3, 0.4 * N, 1e-6)
    assert host(ctx.next_step(to_dev(d), 1.0, 0.3, 0.4 * N)[0])[0] == ref["next"]
    d = inputs.potentials(5, N, scale=40.0)
    assert host(ctx.next_step(to_dev(d), 1.0, 0.3, 2.0 * N)[0])[0] == 0.3 + 1e-6
    assert host(ctx.next_step(to_dev(d), 1.0, 0.3, 0.0)[0])[0] == 1.0
    assert host(ctx.next_step(to_dev(d), 0.0, 0.3, 0.5 * N)[0])[0] == 1.0
    d[N // 3] = np.nan
    assert np.isnan(host(ctx.next_step(to_dev(d), 1.0, 0.3, 0.5 * N)[0])).all()
