"""Performance cases of the burn: what a user's program has this library do.

A hydro code owns zone states in GPU memory and has them burned over its time step, box by box
or all at once; a service submits burns from host memory.  The networks, temperatures, tolerances
and options are those of this repository's benchmark and tests:

  robertson           3 variables, per-zone rate scales, t = 0..1e5
  nv14                13 species + T, 30 reactions, T uniform on 1000..5000 K
  nv14b, nv22, nv48   the networks of the four-network batch, T log-uniform on 90..2500 K
  nv8, nv12, nv20, nv37, nv40   sizes between the kernels' row counts

A case is a dict:
  entry       "burn" (one call), "noalloc" (the allocation-free call), "graph" (replay of a
              captured burn), "batch" (four networks in one call), "server" (requests through
              the continuous-batching server, host data in and out)
  net, zones  network and zones ("batch": total zones, split 4:2:1:1; "server": largest request)
  precision   "fp64", "mixed" (FP32 LU)
  integrator  "bdf", "bdf_variable", "rkc";  reuse: the VODE-style Jacobian and LU reuse
  rtol        tolerance (atol is rtol / 1e4);  source: a constant source per zone;
  retry       zone-by-zone retry after a 1500-step cap
"""
import math

import numpy as np
import torch

from paper_2608_06466_amd import workloads as W
from paper_2608_06466_amd import zoneburn as zb

# species, reactions, seed
RANDOM = {"nv8": (7, 12, 881), "nv12": (11, 25, 615), "nv14": (13, 30, 201), "nv14b": (13, 20, 301),
          "nv20": (19, 40, 616), "nv22": (21, 50, 302), "nv37": (36, 110, 617), "nv40": (39, 120, 612),
          "nv48": (47, 150, 303)}
# step attempts a zone takes, mean over the network's zone distribution at rtol 1e-8
ATTEMPTS = {"robertson": 770, "nv8": 800, "nv12": 600, "nv14": 1987, "nv14b": 570, "nv20": 900,
            "nv22": 1060, "nv37": 1100, "nv40": 1100, "nv48": 1260}
BATCH = ("robertson", "nv14b", "nv22", "nv48")
# largest zone count drawn
MOST = {"robertson": 1 << 20, "nv8": 1 << 17, "nv12": 1 << 17, "nv14": 1 << 17, "nv14b": 1 << 18,
        "nv20": 1 << 16, "nv22": 1 << 16, "nv37": 1 << 13, "nv40": 1 << 13, "nv48": 1 << 13}


def case(name=None, entry="burn", net="nv14", zones=512, precision="fp64", integrator="bdf",
         reuse=False, rtol=1e-8, source=False, retry=False):
    c = dict(entry=entry, net=net, zones=zones, precision=precision, integrator=integrator,
             reuse=reuse, rtol=rtol, source=source, retry=retry)
    return dict(c, name=name) if name else c


def listed():
    return [
        # a few zones left over on a refined patch, replayed as a graph every step: latency
        case("robertson_33_graph", entry="graph", net="robertson", zones=33),
        # the textbook stiff test, one 16^3 box
        case("robertson_4096", net="robertson", zones=4096),
        # a rank's whole level of a small network, ragged
        case("robertson_1m_mixed", net="robertson", zones=1_000_003, precision="mixed"),
        # one 8^3 box inside a loop that must not allocate: a few zones a compute unit
        case("nv14_box8_noalloc", entry="noalloc", zones=512),
        # FP64 throughout, an odd number of zones
        case("nv14_50021_fp64", zones=50_021),
        # the headline workload at a quarter of its zones (one 64^3 box)
        case("nv14_2p18_mixed", zones=1 << 18, precision="mixed"),
        # VODE's own configuration: variable coefficients with Jacobian and LU reuse
        case("nv14_30011_vode_mixed", zones=30_011, precision="mixed", integrator="bdf_variable",
             reuse=True),
        # the middle network, from cold zones of ten steps to hot ones of thousands
        case("nv22_40009_mixed", net="nv22", zones=40_009, precision="mixed"),
        # the largest network: a zone fills a wavefront
        case("nv48_16384_mixed", net="nv48", zones=16_384, precision="mixed"),
        # the largest network at the looser tolerance, with the hydro's constant source
        case("nv48_4099_fp64_source", net="nv48", zones=4_099, rtol=1e-6, source=True),
        # four networks in one call, FP64
        case("batch4_32768_fp64", entry="batch", net="robertson", zones=32_768),
        # requests of mixed networks and sizes from host memory
        case("server_8192_mixed", entry="server", net="robertson", zones=8_192, precision="mixed"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    entry = rng.choice(["burn"] * 6 + ["noalloc", "graph", "batch", "server"])
    precision = rng.choice(["fp64", "mixed"])
    if entry == "batch":
        return case(entry=entry, net="robertson", zones=_log_int(rng, 64, 40_000), precision=precision)
    if entry == "server":
        return case(entry=entry, net="robertson", zones=_log_int(rng, 256, 8_000), precision=precision)
    net = rng.choice(["robertson"] + sorted(RANDOM))
    if net == "nv8":
        precision = "fp64"   # a few of its zones need the FP64 LU
    integrator, reuse, retry = "bdf", False, False
    style = rng.choice(["plain"] * 4 + ["reuse", "variable", "vode", "rkc", "retry"])
    if style in ("reuse", "vode"):
        reuse = True
    if style in ("variable", "vode"):
        integrator = "bdf_variable"
    if style == "rkc" and net in ("nv14b", "nv22", "nv48"):
        integrator, precision = "rkc", "fp64"
    if style == "retry" and net == "nv14":
        retry = True
    return case(entry=entry, net=net, zones=_log_int(rng, 16, MOST[net]), precision=precision,
                integrator=integrator, reuse=reuse, rtol=rng.choice([1e-6, 1e-8, 1e-8]),
                source=net != "robertson" and integrator != "rkc" and rng.random() < 0.2, retry=retry)


def _network(net):
    if net == "robertson":
        return W.robertson_network()
    return W.random_network(*RANDOM[net])


def _zones(net, desc, zones, seed, cold=False):
    """(state, rate scales or None, dt) of fresh zones, host arrays."""
    if net == "robertson":
        state, scale = W.robertson_zones(zones, seed)
        return state, scale, 1.0e5
    if net == "nv14":
        return W.random_zones(desc, zones, seed), None, 1.0
    # RKC is for mildly stiff zones: the cold end of the range
    T = (100.0, 300.0) if cold else W.BATCHED_T_RANGE
    return W.random_zones(desc, zones, seed, T_range=T, T_dist="loguniform"), None, 1.0


def _parts(c):
    """(network name, zones, rtol) of each segment or request of a case."""
    n = c["zones"]
    if c["entry"] == "batch":
        return [(k, max(1, n * w // 8), c["rtol"]) for k, w in zip(BATCH, (4, 2, 1, 1))]
    if c["entry"] == "server":
        sizes = (n, n // 2, n // 4, n // 16, n // 2 + 1, n // 3)
        nets = ("robertson", "nv14b", "nv22", "nv48", "nv14b", "robertson")
        return [(k, max(1, z), c["rtol"] * (100.0 if i % 2 else 1.0))
                for i, (k, z) in enumerate(zip(nets, sizes))]
    return [(c["net"], n, c["rtol"])]


def prepare(c, seed):
    """Context, networks and zone states in hand; for "graph" the captured burn, for "server" the
    running server."""
    ctx = zb.Context(0)
    opts = dict(precision=c["precision"], integrator=c["integrator"],
                jac_policy="reuse" if c["reuse"] else "every_step")
    if c["retry"]:
        opts.update(max_steps=1500, retry=(1e-6, 1e-10, 100000))
    host = c["entry"] == "server"
    segs, nets = [], {}
    for i, (net, zones, rtol) in enumerate(_parts(c)):
        desc = _network(net)
        if net not in nets:
            nets[net] = zb.Network(ctx, desc)
        state, scale, dt = _zones(net, desc, zones, seed * 64 + i, cold=c["integrator"] == "rkc")
        s = dict(net=nets[net], dt=dt, rtol=rtol, atol=rtol * 1e-4)
        if host:
            s.update(input=state, rate_scale=scale)
        else:
            s.update(input=torch.tensor(state, device="cuda:0"),
                     rate_scale=None if scale is None else torch.tensor(scale, device="cuda:0"))
            s["state"] = torch.empty_like(s["input"])
            if c["source"]:
                rng = np.random.default_rng(seed + 5)
                src = np.zeros_like(state)
                src[:, :-1] = rng.uniform(0.0, 1e-3, src[:, :-1].shape)
                src[:, -1] = rng.uniform(-5.0, 5.0, zones)
                s["source"] = torch.tensor(src, device="cuda:0")
            if c["entry"] != "burn":
                s["status"] = torch.empty(zones, dtype=torch.int32, device="cuda:0")
                s["stats"] = torch.empty((zones, 7), dtype=torch.int32, device="cuda:0")
        segs.append(s)
    st = dict(entry=c["entry"], ctx=ctx, nets=nets, segs=segs, opts=opts)
    if host:
        st["server"] = zb.Server(ctx, 256 << 20, **opts)
    if c["entry"] == "graph":
        st["graph"] = zb.Graph(ctx, segs, **opts)
    return st


def run(st):
    segs, opts, entry = st["segs"], st["opts"], st["entry"]
    if entry == "server":
        srv = st["server"]
        tickets = [srv.submit(s["net"], s["input"], s["dt"], s["rtol"], s["atol"], s["rate_scale"])
                   for s in segs]
        out = []
        for t in tickets:
            while not srv.wait(t, timeout=1.0):
                pass
            state, status, stats, _ = srv.fetch(t)
            out.append(dict(state=state, status=status, stats=stats))
        return out
    for s in segs:
        s["state"].copy_(s["input"])   # the burn works in place
    if entry == "burn":
        s = segs[0]
        status, stats = zb.burn(st["ctx"], s["net"], s["state"], s["dt"], s["rtol"], s["atol"],
                                rate_scale=s["rate_scale"], source=s.get("source"), **opts)
        return [dict(state=s["state"], status=status, stats=stats)]
    if entry == "graph":
        st["graph"].launch()
    elif entry == "noalloc":
        zb.burn_batch_noalloc(st["ctx"], segs, **opts)
    else:
        zb.burn_batch(st["ctx"], segs, **opts)
    return [dict(state=s["state"], status=s["status"], stats=s["stats"]) for s in segs]


def work(c):
    """State row in and out, rate scales and source in, status and counters out; per step attempt
    the arithmetic of prediction, norms, one Jacobian, one LU and two Newton iterations (no LU
    or Jacobian solves with RKC)."""
    nbytes = flops = 0.0
    for net, zones, rtol in _parts(c):
        ns, nr = (3, 3) if net == "robertson" else RANDOM[net][:2]
        nv = ns if net == "robertson" else ns + 1
        row = 8 * (ns + 1)
        nbytes += zones * (2 * row + 4 + 28 + (8 * nr if net == "robertson" else 0)
                           + (row if c["source"] else 0))
        newton = 12.0 * nr + 2.0 * nv * nv + 6.0 * nv
        lu = 2.0 * nv ** 3 / 3.0 - nv * nv / 2.0 - nv / 6.0
        attempt = 39.0 * nv + 25.0 * nr + nv * nv + lu + 2.0 * newton
        n = ATTEMPTS[net] * (0.4 if rtol > 1e-7 else 1.0)
        if c["integrator"] == "rkc":
            n, attempt = 60.0, 25.0 * nr + 5.0 * (12.0 * nr + 10.0 * nv)
        flops += zones * n * attempt
    return {"bytes": nbytes, "flops": flops}


def exact(c, seed):
    """Robertson's equations by the three-stage Radau IIA method on a graded mesh fine enough for
    64 bits; None for the other networks and for many zones, where that takes too long."""
    if c["net"] != "robertson" or c["entry"] in ("batch", "server") or c["zones"] > 128:
        return None
    state, scale, dt = _zones("robertson", None, c["zones"], seed * 64)
    k = np.array(W.ROBERTSON_K) * scale
    y = state[:, :3].copy()
    z = len(y)
    s6 = math.sqrt(6.0)
    A = np.array([[(88 - 7 * s6) / 360, (296 - 169 * s6) / 1800, (-2 + 3 * s6) / 225],
                  [(296 + 169 * s6) / 1800, (88 + 7 * s6) / 360, (-2 - 3 * s6) / 225],
                  [(16 - s6) / 36, (16 + s6) / 36, 1.0 / 9.0]])

    def f(u):
        w1, w2, w3 = (k[:, 0] * u[..., 0], k[:, 1] * u[..., 1] ** 2, k[:, 2] * u[..., 1] * u[..., 2])
        return np.stack([w3 - w1, w1 - w2 - w3, w2], axis=-1)

    def jac(u):
        J = np.zeros((z, 3, 3))
        b, d = 2.0 * k[:, 1] * u[:, 1], k[:, 2]
        J[:, 0, 0], J[:, 0, 1], J[:, 0, 2] = -k[:, 0], d * u[:, 2], d * u[:, 1]
        J[:, 1, 0], J[:, 1, 1], J[:, 1, 2] = k[:, 0], -b - d * u[:, 2], -d * u[:, 1]
        J[:, 2, 1] = b
        return J

    mesh = np.concatenate([[0.0], np.geomspace(1e-9, dt, 1500)])
    for t0, t1 in zip(mesh[:-1], mesh[1:]):
        h = t1 - t0
        J = jac(y)
        M = np.eye(9) - h * np.einsum("ij,zkl->zikjl", A, J).reshape(z, 9, 9)
        Minv = np.linalg.inv(M)
        Z = np.zeros((z, 3, 3))
        for _ in range(8):
            F = np.stack([f(y + Z[:, i]) for i in range(3)], axis=1)
            r = (h * np.matmul(A, F) - Z).reshape(z, 9, 1)
            d = np.matmul(Minv, r).reshape(z, 3, 3)
            Z = Z + d
            if np.abs(d).max() < 1e-17:
                break
        y = y + Z[:, 2]
    out = state.copy()
    out[:, :3] = y
    return [dict(state=out, status=None, stats=None)]
