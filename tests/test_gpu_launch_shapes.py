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


@pytest.mark.parametrize("precision", [P.FP64, P.MIXED])
@pytest.mark.parametrize("n1,n2,n7", [(1, 0, 0), (3, 4, 1), (16384, 1, 2), (9001, 8003, 0), (140001, 17, 3)])
def test_batch_of_the_smallest_levels(precision, n1, n2, n7):
    """h = 1/2 and 1/4 in a launch of their own, beside h = 1/128: each item equals
    its single forward (the same solve of each particle, with its status: in the
    mixed form not every particle of these two levels reaches the tolerance)."""
    device()
    case(f"batch precision={precision} h=1/2: {n1}, 1/4: {n2}, 1/128: {n7}")
    c = P.Context(1, 7, 8, 1.0, 0.3, 4, 0.01, precision=precision)
    items = []
    for q, (l, N) in enumerate([(1, n1 // 2), (2, n2), (7, n7), (1, n1 - n1 // 2)]):
        th = to_dev(inputs.theta_batch(40 + q, max(N, 1), 8)[:N])
        items.append(dict(l=l, theta=th, G_out=torch.full((N, 16), np.nan, dtype=torch.float64, device="cuda:0"),
                          status_out=torch.full((N,), -1, dtype=torch.int8, device="cuda:0")))
    for _ in range(2):  # the hand-out counter resets itself
        P.mls2mc_forward_batch(c.h, items)
    for it in items:
        if it["theta"].shape[0] == 0:
            continue
        G, st, _ = c.forward(it["l"], it["theta"], True)
        st, good = host(st), host(st) == 0
        np.testing.assert_array_equal(host(it["status_out"]), st)
        assert good.mean() > 0.9
        assert rel_err(host(it["G_out"])[good], host(G)[good]) < 1e-11
    c.close()


def test_autotuners_name_for_the_resident_solver_with_the_field():
    """{0, 1024, 0, 0} at h = 1/128 is the library's own choice: a launch that
    returns the field takes the same shape as with nothing set, so the same
    device memory and bitwise the same results."""
    device()
    l, N = 7, 1024
    case(f"h=1/128 FP64 field N={N}, default block named")
    G, p = torch.empty((N, 16), dtype=torch.float64, device="cuda:0"), None
    kap = to_dev(_kappa(5, 4, l)).repeat(N // 4, 1)
    out, used = [], []
    for shape in ((0, 0, 0, 0), (0, 0, 0, 0), (0, 1024, 0, 0)):  # the first for the runtime's own allocations
        c = P.Context(l, l, 4, 1.0, 0.3, 4, 0.01)
        c.set_launch(l, *shape)
        p = torch.empty((N, P.mls2mc_ctx_n_unknowns(c.h, l)), dtype=torch.float64, device="cuda:0")
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        P.mls2mc_forward_field(c.h, l, kap, G, p)
        torch.cuda.synchronize()
        used.append(before - torch.cuda.mem_get_info()[0])
        out.append((G.clone(), p[:8].clone()))
        c.close()
    assert used[2] == used[1], used
    assert torch.equal(out[1][0], out[2][0]) and torch.equal(out[1][1], out[2][1])


@pytest.mark.parametrize("precision", [P.FP64, P.MIXED])
def test_lds_budget_of_the_walking_workgroups(precision):
    """1024 threads at V(1,1) from h = 1/256 on: the budget changes nothing, and
    the autotuner does not return one for them."""
    device()
    case(f"h=1/256 precision={precision}: budgets of 1024 threads")
    c = P.Context(8, 8, 4, 1.0, 0.3, 4, 0.01, precision=precision)
    th = to_dev(inputs.theta_batch(60, 5, 4))
    G = []
    for lds in (0, -1, 65536, 81920):
        c.set_launch(8, 4, 1024, 1, lds)
        G.append(c.forward(8, th))
    assert all(torch.equal(G[0], g) for g in G[1:])
    _, (grid, block, nu, lds) = c.autotune(8, 24)
    assert block != 1024 or nu != 1 or lds == 0
    c.close()
