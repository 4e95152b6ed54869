"""Parity of the simulator of models with one gated stage (control state in registers) at
the edges of its range: 64 and 65 members of an iteration, running sets over several pages
of 64 lanes, thinker and talker on one executor and on two, types that use only one of the
two stages, types that use both without the streaming edge between them (so that a talker's
running set holds gated and ungated requests), prefill-only stages, several parents (two
deliveries of a request due together), no transfer delay, CPU preprocessing, tensor-parallel
multipliers, nodes of two configurations, 64 executors, trace lengths around the 64-request
arrival blocks; and a gated model with a third LLM, which the general kernel takes.  Counts,
request-events, status and every latency equal the oracle's bit for bit.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import oracle as O  # noqa: E402
from paper_2512_14098_amd.inputs import plan_table_from_list  # noqa: E402
from tests.helpers import comp, model, rtype  # noqa: E402

LN, LO = {"lognormal": [6.0, 0.5]}, {"lognormal": [4.0, 0.7]}
SPEECH = {"lognormal_s": [1.5, 0.6]}


def _omni(comm=0.010, cpu_pre=0.0, third=False, theta=(9, 10)):
    """Two encoders, thinker, talker, vocoder; with `third` the vocoder is an LLM too."""
    comps = [comp("E1", "ENC", [0.002, 1e-5, 0.0], x=["patches"]),
             comp("E2", "ENC", [0.002, 1e-6, 0.0], x=["aud_in_ms"]),
             comp("Th", "LLM", [0.005, 4e-5, 0.0], x=["prompt", "patches", "aud_in_tok"], decode=(0.012, 8e-5)),
             comp("Ta", "LLM", [0.003, 1e-5, 0.0], x=["prompt"], decode=(0.006, 4e-5), n_out="aud_out_tok", gate="Th"),
             comp("V", "LLM", [0.01, 1e-5, 0.0], x=["out"], decode=(0.004, 1e-5)) if third else
             comp("V", "GEN", [0.01, 1e-5, 0.002], x=["aud_out_tok"], batch_cap=8)]
    for c in comps:
        c["tp_scale"] = {"2": 0.6}
    types = [rtype("both", ["E1", "E2", "Th", "Ta", "V"],
                   [("E1", "Th"), ("E2", "Th"), ("Th", "Ta"), ("Ta", "V")], ["Th", "V"], weight=40,
                   slo={"ttft": 1.0, "tpot": 0.1, "media": 9.0}, images={"const": 1}, prompt=LN, out=LO,
                   aud_in=SPEECH, aud_out=SPEECH),
             rtype("say", ["Th", "Ta"], [("Th", "Ta")], ["Th", "Ta"], weight=30, slo={"e2e": 9.0}, prompt=LN, out=LO,
                   aud_out=SPEECH),
             rtype("text", ["Th"], weight=20, slo={"ttft": 0.5, "tpot": 0.05}, prompt={"const": 300}, out={"exp": 90.0}),
             rtype("short", ["E1", "Th"], [("E1", "Th")], ["Th"], weight=10, slo={"e2e": 3.0}, prompt=LN, out={"const": 1},
                   images={"uniform": [1, 3]})]
    return model(comps, types, comm=comm, cpu_pre=cpu_pre, theta=theta)


PATHS = [[0, 1, 2, 3, 4], [2, 3], [2], [0, 2]]


def _plan(nodes, paths=PATHS):
    return dict(nodes=nodes, routes=[[(10, {c: v for v, nd in enumerate(nodes) for c in t if (nd[0] >> c) & 1})]
                                     for t in paths])


PLANS = [_plan([(31, 1, 256, 1)]),
         _plan([(31, 2, 65, 2)]),
         _plan([(7, 1, 64, 1), (8, 1, 256, 1), (16, 1, 8, 1)]),
         _plan([(1, 1, 16, 1), (2, 1, 16, 1), (12, 2, 256, 1), (16, 2, 8, 1)]),
         _plan([(3, 1, 64, 2), (4, 1, 256, 1), (24, 1, 256, 2)]),
         _plan([(19, 2, 16, 1), (4, 2, 16, 1, 1, 256, 2, 4), (8, 1, 130, 1)]),
         _plan([(1, 4, 16, 1), (2, 4, 16, 1), (4, 24, 64, 1), (8, 24, 64, 1), (16, 8, 8, 1)])]



def _solo(comm=0.010, cpu_pre=0.0):
    """Thinker, a generator, talker, vocoder and an encoder: the talker streamed to, alone, after
    the thinker through the generator, beside the thinker, and with one token only."""
    comps = [comp("E", "ENC", [0.002, 1e-5, 0.0], x=["aud_in_ms"]),
             comp("Th", "LLM", [0.005, 4e-5, 0.0], x=["prompt"], decode=(0.012, 8e-5)),
             comp("M", "GEN", [0.004, 1e-5, 0.001], x=["out"], batch_cap=16),
             comp("Ta", "LLM", [0.003, 1e-5, 0.0], x=["prompt"], decode=(0.006, 4e-5), n_out="aud_out_tok", gate="Th"),
             comp("V", "GEN", [0.01, 1e-5, 0.002], x=["aud_out_tok"], batch_cap=8)]
    for c in comps:
        c["tp_scale"] = {"2": 0.6}
    d = dict(prompt=LN, out=LO, aud_out=SPEECH, slo={"ttft": 1.0, "tpot": 0.1, "e2e": 20.0})
    types = [rtype("stream", ["Th", "Ta", "V"], [("Th", "Ta"), ("Ta", "V")], ["Th", "V"], weight=25, **d),
             rtype("speak", ["Ta"], weight=20, **d),
             rtype("echo", ["E", "Ta", "V"], [("E", "Ta"), ("Ta", "V")], ["Ta", "V"], weight=10, aud_in=SPEECH, **d),
             rtype("relay", ["Th", "M", "Ta"], [("Th", "M"), ("M", "Ta")], ["Th", "Ta"], weight=20, **d),
             rtype("beside", ["Th", "Ta"], [], ["Th", "Ta"], weight=15, **d),
             rtype("brief", ["Th", "Ta"], [("Th", "Ta")], ["Th", "Ta"], weight=5, prefill_only=["Ta"], **d),
             rtype("first", ["Th", "M", "Ta"], [("Th", "M"), ("M", "Ta")], ["Ta"], weight=5, prefill_only=["Th"], **d)]
    return model(comps, types, comm=comm, cpu_pre=cpu_pre)


SOLO_PATHS = [[1, 3, 4], [3], [0, 3, 4], [1, 2, 3], [1, 3], [1, 3], [1, 2, 3]]
SOLO_PLANS = [_plan(nodes, SOLO_PATHS) for nodes in (
    [(31, 1, 256, 1)],
    [(10, 2, 65, 1), (21, 1, 16, 2)],
    [(2, 1, 256, 1), (8, 1, 130, 1), (21, 1, 16, 1)],
    [(10, 1, 64, 2), (5, 2, 8, 1), (16, 1, 8, 1)],
    [(7, 2, 16, 1, 1, 256, 2, 4), (24, 2, 64, 1)])]

CASES = [("mixed", _omni(), 640, [0.5, 6.0, 300.0]),
         ("sync", _omni(comm=0.0, cpu_pre=0.003), 257, [3.0, 80.0]),
         ("pre", _omni(cpu_pre=0.003, theta=(1, 2)), 193, [2.0, 60.0]),
         ("block", _omni(), 64, [4.0]),
         ("one", _omni(), 1, [1.0]),
         ("third_llm", _omni(third=True), 193, [3.0, 80.0])]
SOLO_CASES = [("solo", _solo(), 640, [0.5, 8.0, 300.0]),
              ("solo_sync", _solo(comm=0.0, cpu_pre=0.003), 257, [2.0, 60.0])]


@pytest.mark.parametrize("name,mcfg,n,rates", CASES, ids=[c[0] for c in CASES])
def test_parity_at_the_edges(name, mcfg, n, rates):
    check_parity(name, mcfg, PLANS, n, rates)


@pytest.mark.parametrize("name,mcfg,n,rates", SOLO_CASES, ids=[c[0] for c in SOLO_CASES])
def test_talker_without_its_thinkers_stream(name, mcfg, n, rates):
    check_parity(name, mcfg, SOLO_PLANS, n, rates)


def check_parity(name, mcfg, plans, n, rates):
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
    print(f"fine {name}: {P} plans x {K} rates x {S} seeds x {n} requests", flush=True)
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
