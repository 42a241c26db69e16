"""The resident solver of the flow cell runs the general solver's V-cycle down to
h = 1/2: the same iterations, and the same distance to the solution."""
import numpy as np
import pytest
import torch

import oracle
import paper_1709_09763_amd as P
from tests import inputs
from tests.gpu_util import case, device, host, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("l", [3, 4, 5, 6])
def test_same_iterations_and_error_as_the_general_solver(l):
    """The cycles differ in the rounding of the finest level's weights alone
    (FP32 there, 6e-8): a residual norm moves by about that, so an iteration
    count differs only where the norm meets the tolerance to seven digits, and
    the errors that the tolerance leaves, alike in mean, agree to a few per cent
    (5 % over 48 particles)."""
    device()
    case(f"flow cell l={l}: resident against general")
    N, m = 48, 7
    c = P.Context(l, l, 20, 1.0, 0.3, m, 0.01, bc=P.BC_FLOW_CELL)
    kap = c.kl_field(l, to_dev(inputs.theta_batch(70 + l, N, 20)), P.FIELD_KAPPA_F64)
    res = c.forward_field(l, kap, True)
    c.set_launch(l, N, 256, 1, 0)
    gen = c.forward_field(l, kap, True)
    c.close()
    it = [host(q[3]) for q in (res, gen)]
    assert np.abs(it[0] - it[1]).max() <= 1 and (it[0] != it[1]).sum() <= 1, it
    _, p = oracle.flow_forward_kappa(l, m, host(kap), want_p=True)
    p = p.reshape(N, -1)
    err = [(np.abs(host(q[1]) - p).max(1) / np.abs(p).max(1)).mean() for q in (res, gen)]
    print(f"  mean error resident {err[0]:.3e} general {err[1]:.3e}")
    assert err[0] <= 1.05 * err[1]
    assert torch.isfinite(res[0]).all() and int(res[2].max()) == 0
