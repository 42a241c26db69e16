"""The sampler kernels at the sizes where their forms change: the adaptive step
and resampling in one workgroup or in many, the acceptance's rows beyond one
wave."""
import numpy as np
import pytest
import torch

import oracle
import paper_1709_09763_amd as P
from tests import inputs
from tests.gpu_util import case, device, host, rel_err, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    device()
    c = P.Context(3, 4, 100, 1.0, 0.3, 10, 0.01)
    yield c
    c.close()


@pytest.mark.parametrize("N", [256, 257, 512, 513, 1024, 1025, 2048, 2049, 8192, 8193, 65537, (1 << 18) + 3,
                               (1 << 20) + 1])
def test_next_step_sizes(ctx, N):
    """Interior step, right end and smallest step against the oracle.  The
    bisection's step is where ESS crosses the target: a relative error of the
    two sums of about N^(1/2) 2^-53 moves it by that over the slope of log ESS
    in log t (of order one here), so 1e-12 leaves four digits."""
    case(f"next_step N={N}")
    d = inputs.potentials(7 + N, N, scale=40.0)
    for what, dd, cur, tau in (("interior", d, 0.2, N / 2.0), ("end", 1e-6 * d, 0.2, N / 2.0),
                               ("smallest", np.where(np.arange(N) % 2 == 0, 0.0, 1e9), 0.2, 0.9 * N)):
        out3, logw, w = ctx.next_step(to_dev(dd), 1.0, cur, tau, 1e-6)
        o = host(out3)
        ref = oracle.next_step(dd, 1.0, cur, tau, 1e-6)
        assert abs(o[0] - ref["next"]) <= 1e-12 * max(1e-6, ref["next"] - cur), what
        assert abs(o[1] - ref["dlogZ"]) < 1e-11 * max(1.0, abs(ref["dlogZ"])), what
        assert abs(o[2] - ref["ess"]) < 1e-10 * N, what
        assert rel_err(host(w), ref["w"]) < 1e-10, what
        assert np.abs(host(logw) - -(o[0] - cur) * dd).max() <= 1e-12 * np.abs(dd).max(), what
        if what == "end":
            assert o[0] == 1.0
    d[N // 2] = np.inf
    assert np.isnan(host(ctx.next_step(to_dev(d), 1.0, 0.2, N / 2.0)[0])).all()


@pytest.mark.parametrize("N", [255, 256, 257, 1024, 1025, 4095, 4096, 4097, 8193, 70001])
def test_resample_sizes(ctx, N):
    case(f"resample N={N}")
    w = inputs.weights(N, N, spread=3.0, zero_frac=0.2)
    w[0] = max(w[0], 1e-300)
    u = inputs.uniforms53(N + 5, N)
    u[0], u[-1] = 0.0, 1.0 - 2.0 ** -53
    anc = host(ctx.resample(to_dev(w), to_dev(u)))
    np.testing.assert_array_equal(anc, oracle.resample(w, u))
    one = np.zeros(N)
    one[N - 1] = 5e-324
    assert (host(ctx.resample(to_dev(one), to_dev(u))) == N - 1).all()
    for bad_w, bad_u in ((-1.0, None), (np.nan, None), (np.inf, None), (None, 1.0), (None, -0.5)):
        w2, u2 = w.copy(), u.copy()
        if bad_w is not None:
            w2[N // 3] = bad_w
        else:
            u2[N // 3] = bad_u
        assert (host(ctx.resample(to_dev(w2), to_dev(u2))) == -1).all()


@pytest.mark.parametrize("kernel", [P.KERNEL_PCN, P.KERNEL_RWM])
@pytest.mark.parametrize("N", [1, 7, 130])
def test_accept_copies_whole_rows(ctx, kernel, N):
    """K = 100 and 100 observations (rows longer than a wave): accepted
    particles take the proposal and its response, the others keep theirs,
    and the decisions are those of the acceptance rule in FP64."""
    case(f"accept N={N} kernel={kernel}")
    K, s = 100, 0.3 if kernel == P.KERNEL_PCN else 2.38 / 10
    th = to_dev(inputs.theta_batch(3, N, K))
    xi = to_dev(inputs.theta_batch(4, N, K))
    u = to_dev(1.0 - inputs.uniforms53(5, N))
    y = ctx.forward(4, to_dev(inputs.theta_batch(6, 1, K)))[0].contiguous()
    Gl, Gh = ctx.forward(3, th), ctx.forward(4, th)
    pl, ph = ctx.loglik(Gl, y), ctx.loglik(Gh, y)
    assert rel_err(host(ph), 0.5 * ((host(Gh) - host(y)) ** 2).sum(1) / 1e-4) < 1e-14
    prop = (np.sqrt(1 - s * s) if kernel == P.KERNEL_PCN else 1.0) * host(th) + s * host(xi)
    Gln, Ghn = ctx.forward(3, to_dev(prop)), ctx.forward(4, to_dev(prop))
    beta, zeta = 0.05, 0.4
    psi = lambda a, b, t: beta * ((1 - zeta) * a + zeta * b) + (
        0.5 * (t ** 2).sum(1) if kernel == P.KERNEL_RWM else 0.0)
    delta = psi(host(ctx.loglik(Gln, y)), host(ctx.loglik(Ghn, y)), prop) - psi(host(pl), host(ph), host(th))
    want = np.log(host(u)) < -delta
    t2, l2, h2, pl2, ph2 = th.clone(), Gl.clone(), Gh.clone(), pl.clone(), ph.clone()
    acc = host(ctx.pcn_step(3, 4, beta, zeta, s, t2, l2, h2, pl2, ph2, y, xi, u, kernel)).astype(bool)
    np.testing.assert_array_equal(acc, want)
    for got, old, new, tol in ((t2, th, prop, 1e-15), (l2, Gl, host(Gln), 1e-12), (h2, Gh, host(Ghn), 1e-12)):
        g = host(got)
        np.testing.assert_array_equal(g[~acc], host(old)[~acc])
        if acc.any():
            assert rel_err(g[acc], new[acc]) <= tol
