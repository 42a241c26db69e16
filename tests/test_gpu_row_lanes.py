"""The potential and the acceptance at the row lengths where the number of
lanes per particle changes (1, 4, 16, 64)."""
import numpy as np
import pytest

import paper_1709_09763_amd as P
from tests import inputs
from tests.gpu_util import case, device, host, rel_err, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [1, 2, 3, 4, 5, 9])
@pytest.mark.parametrize("N", [1, 67, 1001])
def test_loglik_rows(m, N):
    """Sums of m^2 positive terms in FP64: (m^2 + 3) 2^-53 relative at most."""
    device()
    case(f"loglik rows nobs={m * m} N={N}")
    c = P.Context(3, 3, 1, 1.0, 0.3, m, 0.01)
    g = inputs.rng(100 * m + N)
    G, y = g.standard_normal((N, m * m)), g.standard_normal(m * m)
    phi = host(c.loglik(to_dev(G), to_dev(y)))
    want = 0.5 * (((y - G).astype(np.longdouble) * np.longdouble(1.0 / 0.01)) ** 2).sum(1)
    assert (np.abs(phi - want) <= (m * m + 3) * 2.0 ** -53 * want).all()
    c.close()


@pytest.mark.parametrize("kernel", [P.KERNEL_PCN, P.KERNEL_RWM])
@pytest.mark.parametrize("mode", ["temper", "bridge", "last"])
@pytest.mark.parametrize("K,m,N", [(1, 1, 333), (3, 1, 333), (4, 1, 333), (7, 3, 333), (8, 3, 333), (32, 4, 333),
                                   (33, 4, 333), (8, 3, 32768), (32, 4, 32769), (33, 4, 32769)])
def test_accept_rows(K, m, N, mode, kernel):
    device()
    case(f"accept rows K={K} nobs={m * m} N={N} {mode} kernel={kernel}")
    O, s = m * m, 0.4
    g = inputs.rng(7 * K + m)
    A, E = g.standard_normal((O, K)), g.standard_normal((O, K))
    c = P.Context(3, 4, K, 1.0, 0.3, m, 0.5)
    c.set_linear_model(A, E)
    l_hi, zeta = {"temper": (3, 1.0), "bridge": (4, 0.4), "last": (4, 1.0)}[mode]
    th, xi = inputs.theta_batch(1, N, K), inputs.theta_batch(2, N, K)
    u = 1.0 - inputs.uniforms53(3, N)
    y = to_dev(g.standard_normal(O))
    state = lambda t: [to_dev(t)] + [c.forward(l, to_dev(t)) for l in (3, 4)]
    prop = (np.sqrt(1 - s * s) if kernel == P.KERNEL_PCN else 1.0) * th + s * xi
    old, new = state(th), state(prop)
    for q in (old, new):
        q += [c.loglik(q[1], y), c.loglik(q[2], y)]
    beta = 0.7

    def psi(q, t):
        lo, hi = host(q[3]), host(q[4])
        v = beta * (lo if mode == "temper" else hi if mode == "last" else (1 - zeta) * lo + zeta * hi)
        return v + (0.5 * (t ** 2).sum(1) if kernel == P.KERNEL_RWM else 0.0)

    d = psi(new, prop) - psi(old, th)
    want = np.log(u) < -d
    t2, l2, h2, pl2, ph2 = [q.clone() for q in old]
    acc = host(c.pcn_step(3, l_hi, beta, zeta, s, t2, None if mode == "last" else l2, None if mode == "temper" else h2,
                          None if mode == "last" else pl2, None if mode == "temper" else ph2, y, to_dev(xi), to_dev(u),
                          kernel)).astype(bool)
    # decisions within rounding of the boundary may go either way
    clear = np.abs(np.log(u) + d) > 1e-10
    np.testing.assert_array_equal(acc[clear], want[clear])
    assert clear.mean() > 0.99 and 0 < acc.sum() < N
    used = {"temper": (0, 1, 3), "bridge": range(5), "last": (0, 2, 4)}[mode]
    for q, got in enumerate((t2, l2, h2, pl2, ph2)):
        got, was = host(got), host(old[q])
        np.testing.assert_array_equal(got[~acc], was[~acc])
        if q in used:
            assert rel_err(got[acc], host(new[q])[acc]) <= 1e-12
        else:
            np.testing.assert_array_equal(got, was)
    c.close()
