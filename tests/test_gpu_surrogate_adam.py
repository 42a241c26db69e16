"""Training steps of the surrogate: Adam on the gradient at the current
parameters, with the BF16 weight copies kept in step."""
import numpy as np
import pytest
import torch

import paper_1709_09763_amd as P
from tests import inputs
from tests.gpu_util import case, device, host, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,m,H,B", [(5, 1, 16, 17), (33, 5, 48, 33), (100, 7, 256, 130), (40, 4, 1024, 40)])
def test_training_steps_are_adam_on_the_current_parameters(K, m, H, B):
    """Each step against Adam in FP64 on loss_grad's gradient of the same rows
    at the same parameters, formed by another context whose copies are made
    anew.  Both gradients are FP32 sums of the same B products, in another
    order: an element differs by at most B 2^-24 times the sum of its terms'
    sizes, under 2.5e-4 of the block's root mean square at B = 130 for terms of
    like size.  Where |g| is at least 0.05 of that, the relative error is below
    5e-3 and an Adam step, of size lr, is off by less than 1e-2 lr.  With
    lr = 0.05 a step moves weights of size 0.1 by half of themselves, so a copy
    or a moment of the step before shows."""
    device()
    case(f"surrogate Adam steps K={K} nobs={m * m} H={H} B={B}")
    O = m * m
    c, ref = P.Context(3, 3, K, 1.0, 0.3, m, 0.01), P.Context(3, 3, K, 1.0, 0.3, m, 0.01)
    for q in (c, ref):
        P.mls2mc_surrogate_init(q.h, H, B, 5)
    x, t = to_dev(inputs.theta_batch(1, B, K)), to_dev(3.0 * inputs.theta_batch(2, B, O))
    P.mls2mc_surrogate_add_pairs(c.h, x, t)

    def standard(a):  # in FP64, the statistics rounded to FP32 as the library keeps them
        mu = a.mean(0).float().double()
        sd = a.std(0, unbiased=False).float().double()
        return ((a - mu) / sd).float().double().contiguous()

    xs, ts = standard(x), standard(t)
    n = P.mls2mc_surrogate_n_params(c.h)
    p = torch.empty(n, dtype=torch.float32, device="cuda:0")
    P.mls2mc_surrogate_get_params(c.h, p)
    cuts = np.cumsum([H * K, H, H * H, H, O * H, O])[:-1]
    lr, b1, b2 = 0.05, 0.9, 0.999
    mom, vel = np.zeros(n), np.zeros(n)
    sure = np.ones(n, dtype=bool)
    loss, g = torch.empty(1, dtype=torch.float32, device="cuda:0"), torch.empty(n, dtype=torch.float32, device="cuda:0")
    for step in range(1, 4):
        before = host(p).astype(np.float64)
        P.mls2mc_surrogate_set_params(ref.h, p)
        P.mls2mc_surrogate_loss_grad(ref.h, xs, ts, loss, g)
        gr = host(g).astype(np.float64)
        P.mls2mc_surrogate_train(c.h, 1, B, lr, step)
        P.mls2mc_surrogate_get_params(c.h, p)
        mom = b1 * mom + (1 - b1) * gr
        vel = b2 * vel + (1 - b2) * gr * gr
        want = -lr * (mom / (1 - b1 ** step)) / (np.sqrt(vel / (1 - b2 ** step)) + 1e-8)
        sure &= np.concatenate([np.abs(a) >= 0.05 * np.sqrt(np.mean(a * a)) for a in np.split(gr, cuts)])
        moved = host(p).astype(np.float64) - before
        assert np.abs(moved - want)[sure].max() <= 1e-2 * lr, step
    assert all(b.any() for b in np.split(sure, cuts))  # every block is compared


@pytest.mark.parametrize("K,m,H,B", [(5, 1, 16, 17), (33, 5, 48, 33), (100, 7, 256, 130)])
def test_training_goes_on_alike_after_the_parameters_are_set_to_themselves(K, m, H, B):
    device()
    case(f"surrogate copies kept against made anew K={K} nobs={m * m} H={H} B={B}")
    n = 3 * B + 5
    x, t = to_dev(inputs.theta_batch(11, n, K)), to_dev(inputs.theta_batch(12, n, m * m))
    got = []
    for anew in (False, True):
        c = P.Context(3, 3, K, 1.0, 0.3, m, 0.01)
        P.mls2mc_surrogate_init(c.h, H, n, 5)
        P.mls2mc_surrogate_add_pairs(c.h, x, t)
        p = torch.empty(P.mls2mc_surrogate_n_params(c.h), dtype=torch.float32, device="cuda:0")
        for epoch in range(3):
            P.mls2mc_surrogate_train(c.h, 1, B, 1e-2, epoch)
            P.mls2mc_surrogate_get_params(c.h, p)
            if anew:
                P.mls2mc_surrogate_set_params(c.h, p.clone())
        got.append(p)
    assert torch.equal(*got)
