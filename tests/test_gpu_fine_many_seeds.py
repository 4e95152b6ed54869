"""Phase 3 over a trace whose 8-byte arrays are longer than 4 GiB: more than 2^29 requests
over all seeds.  The trace is three generated seeds repeated, in an order in which the seeds
2^29 requests apart differ, so a request index held in too few bits reads another seed's
requests.  One case per simulator: control state in registers (no gated stage), the same
with one gated stage, the general one with a gated stage and without.  Every seed's counts,
request-events and status equal those of the seed it repeats, which equal the oracle's.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import oracle as O  # noqa: E402
from paper_2512_14098_amd.inputs import plan_table_from_list  # noqa: E402
from tests.test_gpu_fine_gate import _omni, _plan  # noqa: E402
from tests.test_gpu_fine_reg import _plans_two, _two  # noqa: E402

N, BASE = 256, 3
COPIES = (1 << 29) // (N * BASE) + 2  # ends four seeds past 2^29 requests
OMNI = _plan([(7, 1, 64, 1), (8, 1, 256, 1), (16, 1, 8, 1)])
CASES = [("reg", _two(), _plans_two(32)[0], 200.0),
         ("gate", _omni(), OMNI, 30.0),
         ("general_gated", _omni(third=True), OMNI, 30.0),
         ("general", _two(), _plans_two(33)[0], 200.0)]


@pytest.mark.parametrize("name,mcfg,plan,rate", CASES, ids=[c[0] for c in CASES])
def test_trace_over_2_to_29_requests(name, mcfg, plan, rate):
    from paper_2512_14098_amd import cf
    if torch.cuda.mem_get_info()[0] < 48 << 30:
        pytest.skip("the trace takes 24 GB of device memory")
    tab = plan_table_from_list([plan])
    desc, m = cf.model_desc(mcfg), O.make_model(mcfg)
    seeds = list(range(BASE))
    small, _ = cf.cf_trace_gen(desc, seeds, N)
    otr = O.trace_gen(m, seeds, N)
    # short outputs: the simulations, not the index, set the test's time
    for f, hi in (("out", 6), ("aud_out_ms", 400)):
        small.t[f].clamp_(max=hi)
        otr[f] = np.minimum(otr[f], np.asarray(hi, otr[f].dtype))
    S = BASE * COPIES
    assert S * N > 1 << 29
    print(f"many seeds {name}: {S} seeds x {N} requests", flush=True)
    big = cf.DeviceTrace.__new__(cf.DeviceTrace)
    big.n_seeds, big.n_req = S, N
    big.t, big.c = {}, cf.cf_trace()
    big.c.n_seeds, big.c.n_req = S, N
    for f in small.t:
        big.t[f] = small.t[f].repeat(COPIES)
        setattr(big.c, f + "_dev", big.t[f].data_ptr())
    ids = torch.zeros(1, dtype=torch.int32).cuda()
    r = torch.full((1, 1), rate, dtype=torch.float64).cuda()
    got = cf.cf_eval_fine(desc, cf.DevicePlans(tab), ids, r, big)
    want = O.eval_fine(m, tab, np.zeros(1, np.int32), np.full((1, 1), rate), otr)
    for key, w in zip(("met", "cnt", "events", "status"), want):
        g = got[key].cpu().numpy()
        g = g.view(w.dtype).reshape((COPIES, BASE) + g.shape[3:])
        assert np.array_equal(g[0], w[0, 0]), key
        assert np.array_equal(g, np.broadcast_to(g[:1], g.shape)), key
    del big
    torch.cuda.empty_cache()
