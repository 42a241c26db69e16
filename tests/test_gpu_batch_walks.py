"""Fused batches around the number of h = 1/256 particles that gives the
walked levels a launch of their own: each item equals its single forward."""
import pytest
import torch

import paper_1709_09763_amd as P
from tests import inputs
from tests.gpu_util import case, device, host, rel_err, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [P.FP64, P.MIXED])
@pytest.mark.parametrize("n8", [3, 254, 300])
def test_batch_with_walked_levels(precision, n8):
    device()
    case(f"batch walks precision={precision} n8={n8}")
    c = P.Context(2, 9, 8, 1.0, 0.3, 4, 0.01, precision=precision)
    items = []
    for q, (l, N) in enumerate([(7, 9), (8, n8 - 2), (6, 5), (9, 2), (2, 3), (7, 1)]):
        th = to_dev(inputs.theta_batch(90 + q, N, 8))
        items.append(dict(l=l, theta=th, G_out=torch.empty((N, 16), dtype=torch.float64, device="cuda:0"),
                          status_out=torch.full((N,), -1, dtype=torch.int8, device="cuda:0")))
    for _ in range(2):  # the hand-out counter resets itself
        P.mls2mc_forward_batch(c.h, items)
    for it in items:
        assert (host(it["status_out"]) == 0).all()
        # the same cycle on both sides; only the order of the inner products'
        # terms can differ (mixed: bitwise the separate passes)
        assert rel_err(host(it["G_out"]), host(c.forward(it["l"], it["theta"]))) < 1e-11
