"""Factorisation and triangular solves of the one-row-a-lane kernels at the sizes where they can
go wrong: numbers of variables around their 8-step chunks, 16-row blocks and padded sizes, as
linear networks against the oracle and against the matrix exponential."""
import numpy as np
import pytest
import scipy.linalg as sla

import oracle
from parity import check, gated
from paper_2608_06466_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def zbm():
    from paper_2608_06466_amd import zoneburn as zb
    assert torch.cuda.is_available()
    ctx = zb.Context(0)
    yield zb, ctx
    ctx.close()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("ns", [9, 13, 14, 15, 16, 17, 22, 23, 24, 25, 31, 32, 33, 40, 41, 47, 48])
def test_linear_networks_at_the_edges(zbm, ns, precision):
    """Decay chains with branches (rates 1e-2..1e6), every species fed: the burn is expm(K t) y0.
    The bar is the gated 1e-6 that the integrator is held to at rtol 1e-8."""
    zb, ctx = zbm
    net_d = W.linear_network(ns, 40 + ns, k_range=(1e-2, 1e6), density=2.0 / ns)
    rng = np.random.default_rng(ns)
    st = np.zeros((9, ns + 1))
    st[:, :ns] = rng.dirichlet(np.ones(ns), size=9)
    K = np.zeros((ns, ns))
    for (a, _), (c, _), lk in zip(net_d["reactant"], net_d["product"], net_d["lnA"]):
        K[a, a] -= np.exp(lk)
        K[c, a] += np.exp(lk)
    net = zb.Network(ctx, net_d)
    for policy in ("every_step", "reuse"):
        t = torch.tensor(st, device="cuda:0")
        status, stats = zb.burn(ctx, net, t, 1.0, 1e-8, 1e-12, precision=precision, jac_policy=policy)
        assert zb.sync(ctx) == 0
        out = t.cpu().numpy()
        if policy == "every_step":
            check(f"linear nv {ns} {precision}", (out, status.cpu().numpy(), stats.cpu().numpy()),
                  oracle.burn(net_d, st, 1.0, 1e-8, 1e-12), 1e-8, 1e-12, ns)
        ref = st[:, :ns] @ sla.expm(K).T
        for z in range(len(st)):
            assert gated(out[z, :ns], ref[z], 1e-8, 1e-12) < 1e-6, (policy, z)
    net.close()
