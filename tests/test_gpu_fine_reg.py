"""Parity of the simulator that keeps its control state in registers (models without a
gated stage, plans of at most 64 stage instances) at the edges of its range: one plan of
exactly 64 stage instances (and one of 66, which the general kernel takes), members and
running sets over one page of 64 lanes, components with several parents (two deliveries of
a request due together), several outputs, a zero transfer delay, CPU preprocessing,
tensor-parallel multipliers, trace lengths around the 64-request arrival blocks.  Counts,
request-events, status and every latency equal the oracle's bit for bit.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import oracle as O  # noqa: E402
from paper_2512_14098_amd.inputs import plan_table_from_list  # noqa: E402
from tests.helpers import comp, model, rtype  # noqa: E402

LN, LO = {"lognormal": [6.0, 0.5]}, {"lognormal": [5.0, 0.6]}


def _two(comm=0.010, cpu_pre=0.0):
    comps = [comp("E", "ENC", [0.002, 1e-5, 0.0], x=["patches"]),
             comp("L", "LLM", [0.005, 4e-5, 0.0], x=["prompt", "patches"], decode=(0.012, 8e-5))]
    types = [rtype("text", ["L"], weight=20, slo={"ttft": 0.5, "tpot": 0.05}, prompt=LN, out=LO),
             rtype("image", ["E", "L"], [("E", "L")], ["L"], weight=80, slo={"ttft": 0.5, "tpot": 0.05},
                   images={"uniform": [1, 4]}, prompt=LN, out=LO)]
    return model(comps, types, comm=comm, cpu_pre=cpu_pre)


def _join(comm, cpu_pre):
    tp = {"2": 0.6}
    comps = [comp("E1", "ENC", [0.002, 1e-5, 0.0], x=["patches"]),
             comp("E2", "ENC", [0.002, 1e-6, 0.0], x=["aud_in_ms"]),
             comp("L", "LLM", [0.005, 4e-5, 0.0], x=["prompt", "patches", "aud_in_tok"], decode=(0.012, 8e-5)),
             comp("G", "GEN", [0.05, 0.0, 0.02], x=["out"], batch_cap=8)]
    for c in comps:
        c["tp_scale"] = tp
    types = [rtype("both", ["E1", "E2", "L", "G"], [("E1", "L"), ("E2", "L"), ("L", "G")], ["L", "G"], weight=50,
                   slo={"ttft": 1.0, "media": 9.0}, images={"const": 1}, prompt=LN, out=LO,
                   aud_in={"lognormal_s": [1.5, 0.5]}),
             rtype("draw", ["L", "G"], [("L", "G")], ["G"], weight=30, slo={"media": 5.0}, prompt=LN, out={"const": 7},
                   prefill_only=["L"]),
             rtype("text", ["L"], weight=20, slo={"e2e": 6.0}, prompt={"const": 300}, out={"exp": 90.0})]
    return model(comps, types, comm=comm, cpu_pre=cpu_pre)


def _routes(types, nodes):
    return [[(10, {c: v for v, nd in enumerate(nodes) for c in range(4) if (nd[0] >> c) & 1 and c in t})] for t in types]


def _plans_two(n_exec):
    t = [[1], [0, 1]]
    out = []
    for nodes in ([(3, n_exec, 256, 1)], [(1, 2, 16, 1), (2, 1, 256, 1)], [(1, 1, 64, 1), (2, 3, 64, 1)]):
        out.append(dict(nodes=nodes, routes=_routes(t, nodes)))
    return out


def _plans_join():
    t = [[0, 1, 2, 3], [2, 3], [2]]
    out = []
    for nodes in ([(15, 2, 64, 1)], [(1, 1, 16, 1), (2, 1, 16, 1), (4, 1, 256, 2), (8, 2, 8, 1)],
                  [(3, 1, 64, 2), (12, 2, 256, 1)], [(5, 2, 256, 1), (10, 1, 16, 1, 1, 64, 2, 4)]):
        out.append(dict(nodes=nodes, routes=_routes(t, nodes)))
    return out


CASES = [("two64", _two(), _plans_two(32), 700, [1.0, 40.0, 400.0]),
         ("two66", _two(), _plans_two(33), 257, [40.0, 400.0]),
         ("two_sync", _two(comm=0.0, cpu_pre=0.003), _plans_two(4), 129, [2.0, 60.0]),
         ("join", _join(0.010, 0.003), _plans_join(), 640, [0.5, 6.0, 80.0]),
         ("join_sync", _join(0.0, 0.0), _plans_join(), 193, [3.0, 80.0]),
         ("block", _join(0.010, 0.0), _plans_join(), 64, [4.0]),
         ("one", _two(), _plans_two(1), 1, [1.0])]


@pytest.mark.parametrize("name,mcfg,plans,n,rates", CASES, ids=[c[0] for c in CASES])
def test_parity_at_the_edges(name, mcfg, plans, n, rates):
    from paper_2512_14098_amd import cf
    tab = plan_table_from_list(plans)
    desc, m = cf.model_desc(mcfg), O.make_model(mcfg)
    seeds = [3, 4]
    tr, _ = cf.cf_trace_gen(desc, seeds, n)
    otr = O.trace_gen(m, seeds, n)
    P, K, S = tab.P, len(rates), len(seeds)
    r = np.tile(np.asarray(rates, np.float64), (P, 1))
    ids = np.arange(P, dtype=np.int32)
    lat_ids = list(range(P * K * S))
    print(f"fine_reg {name}: {P} plans x {K} rates x {S} seeds x {n} requests", flush=True)
    out = cf.cf_eval_fine(desc, cf.DevicePlans(tab), torch.from_numpy(ids).cuda(), torch.from_numpy(r).cuda(), tr,
                          lat_triples=lat_ids)
    met, cnt, ev, st = O.eval_fine(m, tab, ids, r, otr)
    assert np.array_equal(out["status"].cpu().numpy().view(np.uint32), st) and not st.any()
    assert np.array_equal(out["cnt"].cpu().numpy().view(np.uint32), cnt)
    assert np.array_equal(out["events"].cpu().numpy().view(np.uint64), ev)
    assert np.array_equal(out["met"].cpu().numpy().view(np.uint32), met)
    lat = out["lat"].cpu().numpy()
    for j in lat_ids:
        p, k, s = j // (K * S), (j // S) % K, j % S
        o = O.sim_triple(m, tab, p, float(r[p, k]), otr, s, want_lat=True)
        assert np.array_equal(lat[j], o["lat"]), (name, p, k, s)
