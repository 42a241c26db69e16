"""Calls with more particles than one grid holds at 64 threads each (2^32
threads), one observation and one KL term each."""
import numpy as np
import pytest
import torch

import paper_1709_09763_amd as P
from tests import inputs
from tests.gpu_util import case, device, to_dev

pytestmark = pytest.mark.gpu

N = (1 << 26) + 5
F64 = dict(dtype=torch.float64, device="cuda:0")


def _needs(gib):
    device()
    if torch.cuda.mem_get_info()[0] < gib * 2 ** 30:
        pytest.skip(f"needs {gib} GiB of free device memory")


@pytest.fixture
def ctx():
    device()
    c = P.Context(3, 3, 1, 1.0, 0.3, 1, 0.01)
    yield c
    c.close()
    torch.cuda.empty_cache()


def test_loglik(ctx):
    _needs(8)
    case(f"loglik N={N}")
    G = torch.linspace(-1.0, 1.0, N, **F64)[:, None]
    y = torch.full((1,), 0.25, **F64)
    phi = torch.full((N,), -1.0, **F64)
    P.mls2mc_loglik(ctx.h, G, y, phi)
    want = 0.5 * ((y - G[:, 0]) * (1.0 / 0.01)) ** 2
    assert torch.allclose(phi, want, rtol=1e-15, atol=0.0)


def test_pcn_step(ctx):
    """G = theta, y = 0, u = 1: a proposal is accepted where it is the smaller
    of the two, which every other one is made to be."""
    _needs(16)
    case(f"pcn_step N={N}")
    ctx.set_linear_model(np.ones((1, 1)), np.zeros((1, 1)))
    th = torch.ones((N, 1), **F64)
    G, y = th.clone(), torch.zeros(1, **F64)
    phi = torch.full((N,), 0.5 / 0.01 ** 2, **F64)
    xi = torch.full((N, 1), 10.0, **F64)
    xi[::2] = -1.0
    acc = torch.full((N,), 7, dtype=torch.uint8, device="cuda:0")
    P.mls2mc_pcn_step(ctx.h, 3, 3, 0.5, 1.0, 0.5, th, G, None, phi, None, y, xi, torch.ones(N, **F64), acc)
    small = np.sqrt(0.75) - 0.5
    assert int(acc[::2].min()) == 1 and int(acc[1::2].max()) == 0
    for a in (th, G):
        assert torch.allclose(a[::2], torch.full_like(a[::2], small), rtol=1e-14)
        assert bool((a[1::2] == 1.0).all())
    assert torch.allclose(phi[::2], torch.full_like(phi[::2], 0.5 * (small / 0.01) ** 2), rtol=1e-12)


def test_surrogate_predict(ctx):
    _needs(8)
    case(f"surrogate_predict N={N}")
    P.mls2mc_surrogate_init(ctx.h, 16, 16, 5)
    x = to_dev(inputs.theta_batch(3, 4096, 1))
    few = torch.empty((4096, 1), **F64)
    P.mls2mc_surrogate_predict(ctx.h, x, few)
    many = x.repeat(N // 4096 + 1, 1)[:N].contiguous()
    G = torch.full((N, 1), float("nan"), **F64)
    P.mls2mc_surrogate_predict(ctx.h, many, G)
    assert torch.equal(G, few.repeat(N // 4096 + 1, 1)[:N])


@pytest.mark.parametrize("bc", [P.BC_DIRICHLET, P.BC_FLOW_CELL])
def test_forward_field(bc):
    _needs(100)
    case(f"forward_field h=1/8 N={N} bc={bc}")
    c = P.Context(3, 3, 1, 1.0, 0.3, 1, 0.01, bc=bc)
    few = c.kl_field(3, to_dev(inputs.theta_batch(4, 1024, 1)), P.FIELD_KAPPA_F64)
    want = c.forward_field(3, few)
    kappa = torch.empty((N, few.shape[1]), **F64)
    block = few.repeat(1024, 1)
    for q in range(0, N, block.shape[0]):
        kappa[q:q + block.shape[0]] = block[:N - q]
    G, _, st, it = c.forward_field(3, kappa)
    for a, b in zip((G, st, it), (want[0], want[2], want[3])):
        assert torch.equal(a[:1024], b) and torch.equal(a[-1029:], torch.cat([b, b[:5]]))
        assert torch.equal(a[(1 << 22) - 1024:(1 << 22) + 1024], torch.cat([b, b]))
    assert int(st.max()) == 0 and bool((G > 0).all())
    c.close()
    del kappa, block
    torch.cuda.empty_cache()
