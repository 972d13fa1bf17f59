"""The lanes per zone chosen when the caller does not: a zone's LDS area grows with its reactions,
and the group widens where two waves of the kernels would no longer fit a CU; a saved tuning file
decides where it was timed on the same kernels."""
import numpy as np
import pytest

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


# The last number of reactions on 16 lanes, four zones a wave in 80 KiB: 2560 doubles a zone, of
# which 246 (330 with the history copy in LDS, FP64) do not grow, and 5 a reaction.
@pytest.mark.parametrize("precision,nr,lanes", [
    ("fp64", 446, 16), ("fp64", 447, 32), ("fp64", 455, 32), ("fp64", 463, 32),
    ("mixed", 446, 16), ("mixed", 462, 16), ("mixed", 463, 16), ("mixed", 464, 32)])
@pytest.mark.parametrize("ns", [9, 13])
def test_lanes_of_a_network_with_many_reactions(zbm, ns, precision, nr, lanes):
    zb, ctx = zbm
    net = zb.Network(ctx, W.random_network(ns, nr, 3))
    assert zb.get_mapping(ctx, net, precision) == lanes
    net.close()


@pytest.mark.parametrize("opts", [dict(), dict(jac_policy=1), dict(integrator="bdf_variable")])
def test_fp64_burn_takes_the_wider_mapping(zbm, opts):
    """455 reactions on 14 variables: the burn without a mapping is bit by bit the one on 32
    lanes, for every method."""
    zb, ctx = zbm
    net_d = W.random_network(13, 455, 3)
    st = W.random_zones(net_d, 19, 6, T_range=(90.0, 200.0), T_dist="loguniform")
    scale = np.exp(np.random.default_rng(3).normal(0.0, 0.3, (19, 455)))
    net = zb.Network(ctx, net_d)
    out = []
    for lanes in (0, 32):
        t = torch.tensor(st, device="cuda:0")
        status, stats = zb.burn(ctx, net, t, 1e-3, 1e-8, 1e-12, lanes=lanes,
                                rate_scale=torch.tensor(scale, device="cuda:0"), **opts)
        assert zb.sync(ctx) == 0
        out.append([x.cpu().numpy() for x in (t, status, stats)])
    for a, b in zip(*out):
        assert np.array_equal(a, b)
    net.close()


def test_tuning_file_of_other_kernels_applies_nothing(zbm, tmp_path):
    """A saved file names the kernels it was timed on; one that names others, or none, leaves the
    context's choices as they are."""
    import json
    zb, _ = zbm
    a = zb.Context(0)
    path = tmp_path / "tune.json"
    zb.tune_save(a, path)
    doc = json.loads(path.read_text())
    doc["entries"] = [{"nv": 14, "nr": 30, "precision": 1, "lanes": 8, "auto_lanes": 8, "auto_lu": 0}]
    net = zb.Network(a, W.nv14_network())
    for kernels, applied in (("0" * 16, 0), (None, 0), (doc["kernels"], 1)):
        other = {k: v for k, v in doc.items() if k != "kernels"}
        if kernels:
            other["kernels"] = kernels
        path.write_text(json.dumps(other))
        assert zb.get_mapping(a, net, "mixed") == 16
        assert zb.tune_load(a, path) == applied
    assert zb.get_mapping(a, net, "mixed") == 8
    net.close()
    a.close()
