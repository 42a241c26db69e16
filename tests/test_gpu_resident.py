"""The register-resident solver of the small levels (h = 1/8 ... 1/64 with the
library's own launch choice) against the oracle and against the general
solvers, which an explicit launch shape selects."""
import numpy as np
import pytest
import torch

import oracle
import paper_1709_09763_amd as P
from oracle import flowcell as fc
from tests import inputs
from tests.gpu_util import case, device, host, rel_err, to_dev

pytestmark = pytest.mark.gpu

FORMS = {"fp64": {}, "mixed": dict(precision=P.MIXED), "flow": dict(bc=P.BC_FLOW_CELL)}


@pytest.mark.parametrize("form", list(FORMS))
@pytest.mark.parametrize("l,N,m,spread", [(3, 1, 3, 1.0), (3, 67, 32, 1.0), (4, 5, 32, 2.5), (5, 33, 5, 1.0),
                                          (5, 3, 32, 2.5), (6, 1, 7, 2.5), (6, 35, 32, 1.0)])
def test_resident_levels_against_oracle_and_general_solver(form, l, N, m, spread):
    """G and the nodal solution on log-normal coefficients (element by
    element, strong contrast among them), with more observations than threads
    (m = 32), against the direct solvers and, for all particles, against the
    general solver: 1e-10 is the forward parity bar of the FP64 solvers
    (1e-9 at contrast e^{+-7}), 1e-6 that of the mixed one.  In FP64 on the
    Dirichlet problem the two solvers run the same cycle to the same
    tolerance, so their iteration counts differ by at most a few (the flow
    cell's and the mixed form's coarsest solves differ)."""
    device()
    case(f"resident {form} l={l} N={N} m={m} spread={spread}")
    ctx = P.Context(l, l, 4, 1.0, 0.3, m, 0.01, **FORMS[form])
    kap = inputs.kappa_batch(900 + 10 * l + N, N, oracle.n_elem(l), spread=spread)
    if form == "mixed":
        kap = kap.astype(np.float32).astype(np.float64)
    kd = to_dev(kap)
    G, p, st, it = ctx.forward_field(l, kd, want_p=True)
    G0, _, st0, it0 = ctx.forward_field(l, kd, want_p=False)
    ctx.set_launch(l, 0, 256, 1, 0)
    Gg, pg, stg, itg = ctx.forward_field(l, kd, want_p=True)
    assert (host(st) == 0).all() and (host(st0) == 0).all() and (host(stg) == 0).all()
    np.testing.assert_array_equal(host(G), host(G0))
    np.testing.assert_array_equal(host(it), host(it0))
    tol = 1e-6 if form == "mixed" else 1e-9 if spread > 2 else 1e-10
    assert rel_err(host(G), host(Gg)) < 2 * tol
    assert rel_err(host(p), host(pg)) < 2 * tol
    if form == "fp64":
        assert np.abs(host(it) - host(itg)).max() <= 4
    idx = [0, N - 1] if N > 1 else [0]
    fwd = fc.forward_kappa if form == "flow" else oracle.forward_kappa
    Gr, pr = fwd(l, m, kap[idx], want_p=True)
    assert rel_err(host(G)[idx], Gr) < tol
    assert rel_err(host(p)[idx], pr) < tol


@pytest.mark.parametrize("form", list(FORMS))
def test_resident_status(form):
    """iteration caps, a non-finite coefficient next to good particles, and
    the independence of a particle's result from its batch"""
    device()
    for l in (3, 4, 5, 6):
        case(f"resident status {form} l={l}")
        ctx = P.Context(l, l, 4, 1.0, 0.3, 5, 0.01, max_iters=3, **FORMS[form])
        kap = inputs.kappa_batch(70 + l, 9, oracle.n_elem(l))
        G, p, st, it = ctx.forward_field(l, to_dev(kap))
        assert (host(st) == 1).all() and (host(it) == 3).all()
        ctx = P.Context(l, l, 4, 1.0, 0.3, 5, 0.01, **FORMS[form])
        bad = kap.copy()
        bad[4, 37] = np.nan
        G, p, st, it = ctx.forward_field(l, to_dev(bad))
        ok = [q for q in range(9) if q != 4]
        assert host(st)[4] == 2 and (host(st)[ok] == 0).all()
        G1, _, st1, it1 = ctx.forward_field(l, to_dev(kap[5:6]))
        np.testing.assert_array_equal(host(G)[5:6], host(G1))


@pytest.mark.parametrize("precision", [P.FP64, P.MIXED])
def test_resident_items_of_a_batch(precision):
    """A fused batch whose levels go to the resident solver, the work-list
    kernel and the exact small levels, in no order and with repeated levels:
    bitwise the single forwards on the resident levels."""
    device()
    case(f"resident batch precision={precision}")
    c = P.Context(2, 7, 12, 1.0, 0.3, 4, 0.01, precision=precision)
    items = []
    for q, (l, N) in enumerate([(4, 3), (7, 5), (6, 17), (3, 70), (2, 2), (6, 1), (5, 9), (4, 64)]):
        th = to_dev(inputs.theta_batch(40 + q, N, 12))
        items.append(dict(l=l, theta=th, G_out=torch.empty((N, 16), dtype=torch.float64, device="cuda:0"),
                          iters_out=torch.empty(N, dtype=torch.int32, device="cuda:0")))
    P.mls2mc_forward_batch(c.h, items)
    for it in items:
        G, st, n = c.forward(it["l"], it["theta"], with_stats=True)
        if 3 <= it["l"] <= 6:
            np.testing.assert_array_equal(host(it["iters_out"]), host(n))
        assert rel_err(host(it["G_out"]), host(G)) < 1e-12
