"""The counters of a zone that is burned up to four times: in mixed precision, that retried, the
FP64 fallback, and that retried."""
import numpy as np
import pytest

from paper_2608_06466_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_retry_with_the_fp64_fallback_sums_every_run():
    """Each zone's row is bitwise that of the run that ended it, and its counters are the sum of
    the plain burns it took: mixed; mixed and its retry; those and the FP64 run; all four (with
    the last one succeeding, and failing).  Without counters the rows and statuses are the same."""
    from paper_2608_06466_amd import zoneburn as zb
    assert torch.cuda.is_available()
    ctx = zb.Context(0)
    net_d = W.random_network(7, 12, 881)
    net = zb.Network(ctx, net_d)
    first, again = (1e-8, 1e-12), (1e-6, 1e-10)

    def run(st, tol, precision, **kw):
        t = torch.tensor(st, device="cuda:0")
        status, stats = zb.burn(ctx, net, t, 1.0, *tol, precision=precision, **kw)
        zb.sync(ctx)
        return t.cpu().numpy(), status.cpu().numpy(), stats.cpu().numpy()

    # zones whose mixed-precision burn and its retry both take many times the FP64 burn's steps
    full = W.random_zones(net_d, 65536, seed=883, T_range=(90.0, 2500.0), T_dist="loguniform")
    slow = [run(full, tol, "mixed", max_steps=6000)[1] != 0 for tol in (first, again)]
    hard = np.nonzero(slow[0] & slow[1])[0][:300]
    assert hard.size >= 10
    st = full[np.union1d(hard, np.arange(300))]
    sf, sa = run(full[hard], first, "fp64"), run(full[hard], again, "fp64")
    assert np.all(sf[1] == 0) and np.all(sa[1] == 0)
    assert max(sf[2][:, 0].max(), sa[2][:, 0].max()) < 6000
    cap1 = int(np.median(sf[2][:, 0]))           # half of them need the FP64 retry,
    need = sa[2][sf[2][:, 0] > cap1, 0]
    cap2 = int(np.quantile(need, 0.7))           # and a third of those fail that too

    m1 = run(st, first, "mixed", max_steps=cap1)
    m2 = run(st, again, "mixed", max_steps=cap2)
    f1 = run(st, first, "fp64", max_steps=cap1)
    f2 = run(st, again, "fp64", max_steps=cap2)
    p1 = m1[1] == 0
    p2 = ~p1 & (m2[1] == 0)
    p3 = ~p1 & ~p2 & (f1[1] == 0)
    p4 = ~p1 & ~p2 & ~p3 & (f2[1] == 0)
    p5 = ~(p1 | p2 | p3 | p4)
    for k, p in enumerate((p1, p2, p3, p4, p5)):
        assert p.sum() > 0, k
    row = np.zeros_like(st)
    status = np.zeros(len(st), np.int32)
    stats = np.zeros((len(st), 7), np.int32)
    for p, r, code, runs in ((p1, m1, 0, (m1,)), (p2, m2, 6, (m1, m2)), (p3, f1, 7, (m1, m2, f1)),
                             (p4, f2, 7, (m1, m2, f1, f2)), (p5, f2, None, (m1, m2, f1, f2))):
        row[p] = r[0][p]
        status[p] = r[1][p] if code is None else code
        stats[p] = sum(x[2][p] for x in runs)

    opts = dict(max_steps=cap1, retry=(*again, cap2), fp64_fallback=True)
    got = run(st, first, "mixed", **opts)
    for a, b in zip(got, (row, status, stats)):
        assert np.array_equal(a, b)
    # no counters asked for
    t = torch.tensor(st, device="cuda:0")
    s = torch.empty(len(st), dtype=torch.int32, device="cuda:0")
    zb.burn_batch(ctx, [dict(net=net, state=t, dt=1.0, rtol=first[0], atol=first[1], status=s)],
                  precision="mixed", **opts)
    assert zb.sync(ctx) == p5.sum()
    assert np.array_equal(t.cpu().numpy(), row) and np.array_equal(s.cpu().numpy(), status)
    net.close()
    ctx.close()
