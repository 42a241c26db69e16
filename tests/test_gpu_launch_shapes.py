"""The library's own launch shapes at the particle counts where they change."""
import numpy as np
import pytest
import torch

import oracle
import paper_1709_09763_amd as P
from tests import inputs
from tests.gpu_util import case, device, host, rel_err, to_dev

pytestmark = pytest.mark.gpu


def _kappa(seed, N, l):
    """log-normal coefficients, constant on blocks of 16 x 16 cells"""
    g = inputs.rng(seed)
    n = 1 << l
    b = np.exp(0.8 * g.standard_normal((N, n // 16, n // 16)))
    return np.repeat(np.repeat(b, 16, axis=1), 16, axis=2)[..., None].repeat(2, axis=3).reshape(N, -1)


@pytest.mark.parametrize("per_cu", [1.0, 1.01, 1.5, 1.51])
def test_mixed_h128_around_one_particle_per_cu(per_cu):
    """Both shapes of the mixed form at h = 1/128: the oracle's bar (1e-6), and
    each other's results to the same bar."""
    device()
    l, m = 7, 4
    N = int(np.ceil(per_cu * torch.cuda.get_device_properties(0).multi_processor_count))
    case(f"mixed h=1/128 N={N}")
    c = P.Context(l, l, 4, 1.0, 0.3, m, 0.01, precision=P.MIXED)
    kap = _kappa(3, 8, l)
    dev = to_dev(np.tile(kap, (N // 8 + 1, 1))[:N])
    G, p, st, _ = c.forward_field(l, dev, True)
    assert (host(st) == 0).all()
    ref = oracle.forward_kappa(l, m, kap[:2])
    assert rel_err(host(G)[:2], ref) < 1e-6
    assert torch.equal(G[:8], G[8 * (N // 8) - 8:8 * (N // 8)]) and torch.equal(p[:8], p[8:16])
    c.set_launch(l, 0, 1024, 0, -1)
    G2, p2, _, _ = c.forward_field(l, dev, True)
    assert rel_err(host(G), host(G2)) < 1e-6 and rel_err(host(p), host(p2)) < 1e-6
    c.close()
