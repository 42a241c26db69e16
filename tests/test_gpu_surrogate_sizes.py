"""The surrogate's fused passes at ragged sizes (widths, outputs and batches
that do not fill their 16- and 32-wide tiles) and a width beyond their LDS,
against the same arithmetic in torch: BF16 operands, exact sums."""
import numpy as np
import pytest
import torch

import paper_1709_09763_amd as P
from tests import inputs
from tests.gpu_util import case, device, host, to_dev

pytestmark = pytest.mark.gpu


def _r(a):
    return a.float().to(torch.bfloat16).double()


def _gelu(z):
    cdf = 0.5 * (1.0 + torch.erf(z / np.sqrt(2.0)))
    return z * cdf, cdf + z * torch.exp(-0.5 * z * z) / np.sqrt(2.0 * np.pi)


def _net(p, x, t, D, H, O):
    W1, b1, W2, b2, W3, b3 = torch.split(p.double(), [H * D, H, H * H, H, O * H, O])
    W1, W2, W3 = _r(W1).view(H, D), _r(W2).view(H, H), _r(W3).view(O, H)
    z1 = _r(x) @ W1.T + b1
    h1, d1 = _gelu(z1)
    z2 = _r(h1) @ W2.T + b2
    h2, d2 = _gelu(z2)
    out = _r(h2) @ W3.T + b3
    if t is None:
        return out
    g3 = (out - t) / t.numel()
    g2 = (_r(g3) @ W3) * d2
    g1 = (_r(g2) @ W2) * d1
    return [_r(g1).T @ _r(x), g1.sum(0), _r(g2).T @ _r(h1), g2.sum(0), _r(g3).T @ _r(h2), g3.sum(0)], \
        0.5 * ((out - t) ** 2).mean()


@pytest.mark.parametrize("K,m,H,B", [(1, 1, 16, 1), (5, 1, 16, 17), (33, 5, 48, 33), (100, 7, 256, 130),
                                     (512, 10, 512, 64), (40, 4, 1024, 40)])
def test_surrogate_sizes(K, m, H, B):
    """An operand whose FP32 value lies next to a BF16 rounding boundary can
    round the other way than here (2^-8 of that term), all else is FP32
    rounding: 1e-2 of the block's norm covers a flip in every product chain
    of the smallest blocks and is far below a wrong or missing term."""
    device()
    case(f"surrogate K={K} nobs={m * m} H={H} B={B}")
    O = m * m
    c = P.Context(3, 3, K, 1.0, 0.3, m, 0.01)
    P.mls2mc_surrogate_init(c.h, H, 256, 5)
    n = P.mls2mc_surrogate_n_params(c.h)
    p = torch.empty(n, dtype=torch.float32, device="cuda:0")
    P.mls2mc_surrogate_get_params(c.h, p)
    p += 0.05 * torch.tensor(inputs.rng(3).standard_normal(n), dtype=torch.float32, device="cuda:0")  # biases too
    P.mls2mc_surrogate_set_params(c.h, p)
    x, t = to_dev(inputs.theta_batch(1, B, K)), to_dev(3.0 * inputs.theta_batch(2, B, O))
    loss = torch.empty(1, dtype=torch.float32, device="cuda:0")
    g = torch.empty(n, dtype=torch.float32, device="cuda:0")
    P.mls2mc_surrogate_loss_grad(c.h, x, t, loss, g)
    G = torch.empty((B, O), dtype=torch.float64, device="cuda:0")
    P.mls2mc_surrogate_predict(c.h, x, G)
    ref, L = _net(p.cpu(), x.cpu(), t.cpu(), K, H, O)
    out = _net(p.cpu(), x.cpu(), None, K, H, O)
    assert np.linalg.norm(host(G) - out.numpy()) <= 1e-2 * np.linalg.norm(out.numpy())
    assert abs(host(loss)[0] - float(L)) <= 1e-2 * float(L)
    cuts = np.cumsum([H * K, H, H * H, H, O * H, O])[:-1]
    for a, b in zip(np.split(host(g).astype(np.float64), cuts), ref):
        b = b.numpy().ravel()
        assert np.linalg.norm(a - b) <= 1e-2 * np.linalg.norm(b)
    # parameters set anew are the ones used
    P.mls2mc_surrogate_set_params(c.h, torch.zeros_like(p))
    P.mls2mc_surrogate_predict(c.h, x, G)
    assert host(G).any() == False  # noqa: E712
