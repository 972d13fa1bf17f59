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


def _mixed_orders(ns, seed):
    """Thermal network of one- and two-reactant reactions: every third reaction of a random
    network loses its second reactant and product, every seventh consumes one species twice, every
    fifth has its first reactant among the products."""
    net = W.random_network(ns, 3 * ns, seed, E_range=(1.0e3, 2.0e4))
    ra, pa = net["reactant"], net["product"]
    pa[::5, 0] = ra[::5, 0]
    ra[::7, 1] = ra[::7, 0]
    ra[::3, 1] = pa[::3, 1] = -1
    pa[::3, 0] = (ra[::3, 0] + 1) % ns
    net["lnA"] = net["lnA"] * 0.7
    net["q"] = net["q"] * 1e-3   # the cycles among them would heat without end
    return net


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("ns", [3, 7, 13, 15, 21, 31, 33, 47])
def test_reaction_tables(zbm, ns, precision):
    """The packed reaction and row tables of the evaluation: unary, A + A and catalytic reactions
    on every kernel size, against the oracle's bars at rtol 1e-8."""
    zb, ctx = zbm
    net_d = _mixed_orders(ns, 70 + ns)
    st = W.random_zones(net_d, 21, 71 + ns, T_range=(300.0, 1500.0), T_dist="loguniform")
    net = zb.Network(ctx, net_d)
    t = torch.tensor(st, device="cuda:0")
    status, stats = zb.burn(ctx, net, t, 1.0, 1e-8, 1e-12, precision=precision)
    assert zb.sync(ctx) == 0
    check(f"tables nv {ns + 1} {precision}", (t.cpu().numpy(), status.cpu().numpy(), stats.cpu().numpy()),
          oracle.burn(net_d, st, 1.0, 1e-8, 1e-12), 1e-8, 1e-12, ns + 1,
          fine=oracle.burn(net_d, st, 1.0, 1e-10, 1e-14, max_steps=10000000), state_in=st)
    net.close()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("ns", [4, 13, 48])
def test_no_reactions(zbm, ns, precision):
    """No reactions (padding entries only): every zone ends as it began."""
    zb, ctx = zbm
    net_d = W.random_network(ns, 0, 5, thermal=ns < 48)
    st = W.random_zones(net_d, 5, 6)
    net = zb.Network(ctx, net_d)
    t = torch.tensor(st, device="cuda:0")
    zb.burn(ctx, net, t, 1.0, 1e-8, 1e-12, precision=precision)
    assert zb.sync(ctx) == 0
    assert np.array_equal(t.cpu().numpy(), st)
    net.close()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("nv,lanes", [(6, 16), (8, 16), (12, 32), (16, 32), (24, 64), (40, 64)])
def test_solve_skips_whole_chunks(zbm, nv, lanes, precision):
    """Networks that leave whole 8-step chunks of the kernel's rows unused (8 variables on the
    14-row kernel, 16 on the 22-row one): the solves take the chunks that the LU took, and no
    pivot of a skipped row, which is never set.  Both Jacobian policies, against the oracle."""
    zb, ctx = zbm
    net_d = W.random_network(nv - 1, 2 * nv, 900 + nv)
    st = W.random_zones(net_d, 24, 901 + nv, T_range=(90.0, 1000.0), T_dist="loguniform")
    net = zb.Network(ctx, net_d)
    for policy in (0, 1):
        t = torch.tensor(st, device="cuda:0")
        status, stats = zb.burn(ctx, net, t, 1.0, 1e-8, 1e-12, precision=precision, lanes=lanes,
                                jac_policy=policy)
        assert zb.sync(ctx) == 0
        check(f"nv {nv} on {lanes} lanes {precision} policy {policy}",
              (t.cpu().numpy(), status.cpu().numpy(), stats.cpu().numpy()),
              oracle.burn(net_d, st, 1.0, 1e-8, 1e-12, jac_policy=policy), 1e-8, 1e-12, nv,
              fine=oracle.burn(net_d, st, 1.0, 1e-10, 1e-14, jac_policy=policy, max_steps=10000000), state_in=st)
    net.close()
