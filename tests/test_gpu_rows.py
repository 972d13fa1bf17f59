"""The walk over a species' reaction list at the list lengths where it can go wrong: around the
twelve entries that the 14-row kernels request at once, around whole loads of four entries, and
lists of very unequal length in the kernels that hold several rows a lane."""
import numpy as np
import pytest

import oracle
from parity import check
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


def _list_lengths(net):
    ns = net["n_species"]
    n = np.zeros(ns, int)
    for (a, b), (c, d) in zip(net["reactant"], net["product"]):
        for i in range(ns):
            n[i] += int(c == i) + int(d == i) != int(a == i) + int(b == i)
    return n


def hub_network(ns, longest, seed):
    """Thermal two-body network whose species 0 is in every reaction, consumed by every second
    one: its list has `longest` entries, the others share 3 longest places (little heat, or the
    cycles would run away)."""
    net = W.random_network(ns, longest, seed, E_range=(1.0e3, 2.0e4))
    rng = np.random.default_rng(seed)
    for r in range(longest):
        o = rng.integers(1, ns, size=3)
        net["reactant"][r] = (0, o[0]) if r % 2 else (o[0], o[1])
        net["product"][r] = (o[1], o[2]) if r % 2 else (o[2], 0)
    net["lnA"] = net["lnA"] * 0.7
    net["q"] = net["q"] * 1e-4
    return net


def _parity(zb, ctx, net_d, zones, seed, name, policies=(0, 1), form="fixed", **kw):
    nv = net_d["n_species"] + 1
    if form == "variable":
        kw["integrator"] = "bdf_variable"
    st = W.random_zones(net_d, zones, seed, T_range=(300.0, 1500.0), T_dist="loguniform")
    net = zb.Network(ctx, net_d)
    for policy in policies:
        t = torch.tensor(st, device="cuda:0")
        status, stats = zb.burn(ctx, net, t, 1.0, 1e-8, 1e-12, jac_policy=policy, **kw)
        assert zb.sync(ctx) == 0
        check(f"{name} policy {policy}", (t.cpu().numpy(), status.cpu().numpy(), stats.cpu().numpy()),
              oracle.burn(net_d, st, 1.0, 1e-8, 1e-12, jac_policy=policy, form=form), 1e-8, 1e-12, nv,
              fine=oracle.burn(net_d, st, 1.0, 1e-10, 1e-14, jac_policy=policy, form=form, max_steps=10000000),
              state_in=st)
    net.close()


# (variables, lanes) of the kernels with several rows a lane and, beside them, one row a lane
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("nv,lanes", [(4, 1), (16, 4), (14, 4), (16, 8), (9, 8), (16, 16)])
@pytest.mark.parametrize("longest", [4, 5, 8, 41])
def test_lists_of_unequal_length(zbm, nv, lanes, longest, precision):
    """Rows whose lists end in the first load, at the end of a load, and after many, side by side
    in a lane: each contributes all of its entries."""
    zb, ctx = zbm
    net_d = hub_network(nv - 1, longest, 300 + nv + longest)
    n = _list_lengths(net_d)
    assert n[0] == longest
    _parity(zb, ctx, net_d, 17, 301, f"hub nv {nv} lanes {lanes} longest {longest} {precision}",
            policies=(0,), precision=precision, lanes=lanes)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("ns,longest", [(8, 12), (8, 13), (13, 12), (13, 13), (13, 16), (13, 17), (11, 41)])
def test_lists_around_the_requested_entries(zbm, ns, longest, precision):
    """The 14-row kernels request twelve entries of a row at once and stream longer lists: lists of
    exactly 12, of 13 (the first to stream), whole loads and one more, under both Jacobian
    policies."""
    zb, ctx = zbm
    net_d = hub_network(ns, longest, 400 + ns + longest)
    assert _list_lengths(net_d).max() == longest
    _parity(zb, ctx, net_d, 21, 401, f"list nv {ns + 1} longest {longest} {precision}", precision=precision)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("form", ["fixed", "variable"])
def test_many_reactions_a_species(zbm, form, precision):
    """13 species and 80 reactions, lists of up to 31 entries, in both forms of the integrator and
    under both policies: all four 14-row kernels of a precision stream them."""
    zb, ctx = zbm
    net_d = W.random_network(13, 80, 77, E_range=(1.0e3, 2.0e4))
    net_d["lnA"] = net_d["lnA"] * 0.7
    net_d["q"] = net_d["q"] * 1e-3
    assert _list_lengths(net_d).max() == 31
    _parity(zb, ctx, net_d, 21, 402, f"80 reactions {form} {precision}", form=form, precision=precision)


def _mixed_orders(ns, seed):
    """One- and two-reactant reactions: every third reaction of a random network loses its second
    reactant and product, every seventh consumes one species twice, every fifth has its first
    reactant among the products (little heat, or the cycles would run away)."""
    net = W.random_network(ns, 3 * ns, seed, E_range=(1.0e3, 2.0e4))
    ra, pa = net["reactant"], net["product"]
    pa[::5, 0] = ra[::5, 0]
    ra[::7, 1] = ra[::7, 0]
    ra[::3, 1] = pa[::3, 1] = -1
    pa[::3, 0] = (ra[::3, 0] + 1) % ns
    net["lnA"] = net["lnA"] * 0.7
    net["q"] = net["q"] * 1e-3
    return net


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("ns,policies", [(23, (0, 1)), (3, (1,)), (7, (1,)), (13, (1,)), (15, (1,)), (21, (1,)),
                                         (31, (1,)), (47, (1,))])
def test_reaction_tables_under_reuse(zbm, ns, policies, precision):
    """Unary, A + A and catalytic reactions under the Jacobian reuse on every kernel size, and
    on the 24-row kernels under both policies."""
    zb, ctx = zbm
    _parity(zb, ctx, _mixed_orders(ns, 170 + ns), 21, 171 + ns, f"tables nv {ns + 1} {precision}",
            policies=policies, precision=precision)
