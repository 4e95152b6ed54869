"""The general simulators, which keep their stage table in LDS and take what the ones in
registers do not: k_fine<true> models with a gated stage and a third LLM component,
k_fine<false> launches of models without one in which some plan has more than 64 stage
instances.  Parity with the oracle (counts, request-events, status, latencies, latency
histograms) on plans whose nodes hold one and two configurations, the allocation-free entry
point, and the failure statuses: capacity and instant limits forced from the host, invalid
plans and rates.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import oracle as O  # noqa: E402
from paper_2512_14098_amd.inputs import plan_table_from_list  # noqa: E402
from tests.test_gpu_fine_gate import PLANS as OMNI_PLANS, _omni, check_parity  # noqa: E402
from tests.test_gpu_fine_reg import _join, _plans_join, _routes  # noqa: E402
from tests.test_gpu_status import ST_DEADLOCK, ST_INVALID, ST_OVERFLOW, _check_against_free, _np  # noqa: E402

# 17 executors of four components: 68 stage instances
WIDE = dict(nodes=[(15, 17, 64, 1)], routes=_routes([[0, 1, 2, 3], [2, 3], [2]], [(15, 17, 64, 1)]))
SETS = {"gated": (_omni(third=True, cpu_pre=0.003), OMNI_PLANS, [3.0, 80.0]),
        "ungated": (_join(0.010, 0.003), _plans_join() + [WIDE], [3.0, 80.0])}
BOTH = pytest.mark.parametrize("name", sorted(SETS))


def _stages(plan):
    return sum(bin(nd[0]).count("1") * (nd[1] + (nd[4] if len(nd) > 4 else 0)) for nd in plan["nodes"])


def _launch(name, n, seeds):
    from paper_2512_14098_amd import cf
    mcfg, plans, rates = SETS[name]
    tab = plan_table_from_list(plans)
    desc = cf.model_desc(mcfg)
    tr, _ = cf.cf_trace_gen(desc, seeds, n)
    r = np.tile(np.asarray(rates, np.float64), (tab.P, 1))
    ids = torch.arange(tab.P, dtype=torch.int32).cuda()
    return cf, mcfg, tab, desc, cf.DevicePlans(tab), ids, r, tr


@BOTH
def test_parity(name):
    mcfg, plans, rates = SETS[name]
    if name == "gated":
        assert sum(c["kind"] == "LLM" for c in mcfg["components"]) == 3
    else:
        assert max(_stages(p) for p in plans) > 64
    check_parity("general_" + name, mcfg, plans, 321, rates)


@BOTH
def test_histograms_and_the_allocation_free_entry_point(name):
    n, seeds = 200, [5, 6]
    cf, mcfg, tab, desc, plans, ids, r, tr = _launch(name, n, seeds)
    m = O.make_model(mcfg)
    otr = O.trace_gen(m, seeds, n)
    tg = O.scaled_targets(m, [0.25, 0.5, 1.0, 2.0, 4.0])
    print(f"general {name}: histograms of {tab.P} plans", flush=True)
    rates = torch.from_numpy(r).cuda()
    lat = [0, tab.P * r.shape[1] * 2 - 1]
    out = cf.cf_eval_fine(desc, plans, ids, rates, tr, lat_triples=lat, targets=tg)
    hist = out["hist"].cpu().numpy().view(np.uint32)
    for p in range(tab.P):
        for k in range(r.shape[1]):
            for s in range(2):
                o = O.sim_triple(m, tab, p, float(r[p, k]), otr, s, want_lat=True)
                want = O.latency_hist(o["lat"], otr["type"][s * n:(s + 1) * n], m.n_types, tg)
                assert np.array_equal(hist[p, k, s], want), (p, k, s)
    got = cf.cf_eval_fine_noalloc(desc, plans, ids, rates, tr, lat_triples=lat, targets=tg)
    for key in ("met", "cnt", "events", "status", "lat", "hist"):
        assert torch.equal(got[key], out[key]), key


@BOTH
@pytest.mark.parametrize("key,values,status", [("chunks", [2, 3, 4, 6, 8, 12, 16, 24, 32, 64], ST_OVERFLOW),
                                               ("delay", [2, 4, 8, 16, 32, 64, 128, 256], ST_OVERFLOW),
                                               ("instants", [64, 256, 512, 1024, 2048, 4096, 8192, 16384, 32768], ST_DEADLOCK)],
                         ids=["chunks", "delay", "instants"])
def test_limits(name, key, values, status):
    cf, mcfg, tab, desc, plans, ids, r, tr = _launch(name, 600, [0, 1])
    rates = torch.from_numpy(r).cuda()
    free = _np(cf.cf_eval_fine(desc, plans, ids, rates, tr))
    assert not free["status"].any()
    mixed = 0
    for v in values:
        print(f"general {name}: {key} = {v}", flush=True)
        n_ok, n_bad = _check_against_free(_np(cf.cf_eval_fine(desc, plans, ids, rates, tr, limits={key: v})), free, status)
        mixed += bool(n_ok and n_bad)
    assert mixed  # some limit stops a part of the launch only
    again = _np(cf.cf_eval_fine(desc, plans, ids, rates, tr))
    for f in free:
        assert np.array_equal(again[f], free[f]), f


@BOTH
def test_invalid_plans_and_rates(name):
    n = 100
    cf, mcfg, tab, desc, plans, ids, r, tr = _launch(name, n, [0])
    split = next(p for p in range(tab.P) if np.any(tab.node_rep2[:, p]))
    bad = tab.subset(list(range(tab.P)) + [split])
    bad.node_w[int(np.argmax(bad.node_rep2[:, tab.P] > 0)), tab.P] = 10
    ids = np.array(list(range(tab.P)) + [tab.P, tab.P + 9, -1], np.int32)
    rates = np.tile(np.array([4.0, np.nan, -1.0, 30.0]), (len(ids), 1))
    out = _np(cf.cf_eval_fine(desc, cf.DevicePlans(bad), torch.from_numpy(ids).cuda(), torch.from_numpy(rates).cuda(), tr))
    m = O.make_model(mcfg)
    otr = O.trace_gen(m, [0], n)
    st = out["status"].view(np.uint32)[:, :, 0]
    for i, p in enumerate(ids):
        for k in range(4):
            if i >= tab.P or k in (1, 2):
                assert st[i, k] == ST_INVALID and not out["cnt"][i, k].any(), (i, k)
            else:
                o = O.sim_triple(m, tab, int(p), float(rates[i, k]), otr, 0)
                assert st[i, k] == o["status"] == 0
                assert np.array_equal(out["met"][i, k, 0].view(np.uint32), o["met"]), (i, k)
                assert np.array_equal(out["cnt"][i, k, 0].view(np.uint32), o["cnt"]), (i, k)
