"""The flow cell's fused row walks (h = 1/256 on, V(1,1), blocks that half the
row width divides) against the separate sweeps, which a 64-thread block
selects, and against the oracle."""
import numpy as np
import pytest

import oracle
import paper_1709_09763_amd as P
from oracle import flowcell as fc
from tests import inputs
from tests.gpu_util import case, device, host, rel_err, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("l,N,block,spread", [(8, 2, 0, 1.0), (8, 3, 128, 1.0), (8, 1, 256, 2.5), (8, 2, 512, 1.0),
                                              (9, 1, 0, 1.0), (9, 1, 256, 1.0), (9, 2, 512, 1.0)])
def test_flow_walks_against_separate_sweeps_and_oracle(l, N, block, spread):
    """Every node of the walks evaluates the separate sweeps' expressions, only
    the order of the terms of <r, z> differs: the solutions agree to 1e-11
    (both stop at 1e-11 of the first <r, z>^(1/2)) and the iteration counts to
    one.  1e-10 (1e-9 at contrast e^{+-7}) is the forward parity bar."""
    device()
    case(f"flow walks l={l} N={N} block={block} spread={spread}")
    ctx = P.Context(l, l, 4, 1.0, 0.3, 6, 0.01, bc=P.BC_FLOW_CELL)
    kap = inputs.kappa_batch(300 + l + N, N, oracle.n_elem(l), spread=spread)
    kd = to_dev(kap)
    ctx.set_launch(l, 0, block, 1, 0)
    G, p, st, it = ctx.forward_field(l, kd, want_p=True)
    G0, _, st0, it0 = ctx.forward_field(l, kd, want_p=False)
    ctx.set_launch(l, 0, 64, 1, 0)
    Gs, ps, sts, its = ctx.forward_field(l, kd, want_p=True)
    assert (host(st) == 0).all() and (host(st0) == 0).all() and (host(sts) == 0).all()
    assert rel_err(host(p), host(ps)) < 1e-11
    assert rel_err(host(G), host(Gs)) < 1e-11
    assert rel_err(host(G0), host(G)) < 1e-11
    assert np.abs(host(it) - host(its)).max() <= 1
    if l == 8:
        tol = 1e-9 if spread > 2 else 1e-10
        Gr, pr = fc.forward_kappa(l, 6, kap[:1], want_p=True)
        assert rel_err(host(G)[:1], Gr) < tol
        assert rel_err(host(p)[:1], pr) < tol
