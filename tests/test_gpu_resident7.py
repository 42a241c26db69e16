"""The register-resident solver at h = 1/128 (FP64 Dirichlet, the library's own
launch choice) against the oracle and against the general solver, which an
explicit launch shape, a request for the field or more observations than the
kernel's list holds select."""
import numpy as np
import pytest
import torch

import oracle
import paper_1709_09763_amd as P
from tests import inputs
from tests.gpu_util import case, device, host, rel_err, to_dev

pytestmark = pytest.mark.gpu
L = 7


@pytest.mark.parametrize("N,m,spread", [(1, 3, 1.0), (35, 11, 1.0), (3, 17, 1.0), (3, 7, 2.5), (300, 10, 1.0)])
def test_h128_against_oracle_and_general_solver(N, m, spread):
    """1e-10 is the forward parity bar of the FP64 solvers (1e-9 at contrast
    e^{+-7}); both solvers run the same cycle to the same tolerance, so their
    iteration counts differ by at most a few.  300 particles are more than
    workgroups; 11 x 11 observations are the most on a square grid that the
    list holds."""
    device()
    case(f"resident7 N={N} m={m} spread={spread}")
    ctx = P.Context(L, L, 4, 1.0, 0.3, m, 0.01)
    kap = inputs.kappa_batch(700 + N, N, oracle.n_elem(L), spread=spread)
    kd = to_dev(kap)
    G, _, st, it = ctx.forward_field(L, kd, want_p=False)
    Gp, p, stp, _ = ctx.forward_field(L, kd, want_p=True)
    ctx.set_launch(L, 0, 512, 1, 0)
    Gg, _, stg, itg = ctx.forward_field(L, kd, want_p=False)
    assert (host(st) == 0).all() and (host(stp) == 0).all() and (host(stg) == 0).all()
    tol = 1e-9 if spread > 2 else 1e-10
    assert rel_err(host(G), host(Gg)) < 2 * tol
    assert rel_err(host(G), host(Gp)) < 2 * tol
    assert np.abs(host(it) - host(itg)).max() <= 4
    idx = [0, N - 1] if N > 1 else [0]
    Gr = oracle.forward_kappa(L, m, kap[idx])
    assert rel_err(host(G)[idx], Gr) < tol


def test_h128_status():
    """iteration caps, a non-finite coefficient next to good particles, a
    launch after it, and the independence of a result from its batch"""
    device()
    case("resident7 status")
    ctx = P.Context(L, L, 4, 1.0, 0.3, 5, 0.01, max_iters=3)
    kap = inputs.kappa_batch(77, 9, oracle.n_elem(L))
    G, _, st, it = ctx.forward_field(L, to_dev(kap), want_p=False)
    assert (host(st) == 1).all() and (host(it) == 3).all()
    ctx = P.Context(L, L, 4, 1.0, 0.3, 5, 0.01)
    bad = kap.copy()
    bad[4, 37] = np.nan
    G, _, st, it = ctx.forward_field(L, to_dev(bad), want_p=False)
    ok = [q for q in range(9) if q != 4]
    assert host(st)[4] == 2 and (host(st)[ok] == 0).all()
    for q in (5, 8):
        G1, _, st1, it1 = ctx.forward_field(L, to_dev(kap[q:q + 1]), want_p=False)
        np.testing.assert_array_equal(host(G)[q:q + 1], host(G1))


def test_h128_items_of_a_batch_and_unaligned_coefficients():
    """several items of the level in one batch, bitwise the single forwards;
    coefficients that start at an odd multiple of eight bytes"""
    device()
    case("resident7 batch")
    c = P.Context(5, 8, 12, 1.0, 0.3, 4, 0.01)
    items = []
    for q, (l, N) in enumerate([(7, 3), (5, 4), (7, 290), (8, 2), (7, 1)]):
        th = to_dev(inputs.theta_batch(60 + q, N, 12))
        items.append(dict(l=l, theta=th, G_out=torch.empty((N, 16), dtype=torch.float64, device="cuda:0"),
                          iters_out=torch.empty(N, dtype=torch.int32, device="cuda:0")))
    P.mls2mc_forward_batch(c.h, items)
    for it in items:
        G, st, n = c.forward(it["l"], it["theta"], with_stats=True)
        assert (host(st) == 0).all()
        if it["l"] == L:
            np.testing.assert_array_equal(host(it["iters_out"]), host(n))
            np.testing.assert_array_equal(host(it["G_out"]), host(G))
    kap = inputs.kappa_batch(5, 3, oracle.n_elem(L))
    flat = torch.empty(kap.size + 1, dtype=torch.float64, device="cuda:0")
    off = flat[1:].view(3, -1)
    off.copy_(to_dev(kap))
    G = c.forward_field(L, to_dev(kap), want_p=False)[0]
    G1 = c.forward_field(L, off, want_p=False)[0]
    np.testing.assert_array_equal(host(G), host(G1))
