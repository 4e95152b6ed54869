"""Phase 1's routing shares: whole tenths (tabulated), shares that are no tenths, a share of
zero, one alternative; plan counts about a block's size, few and all batch sizes, invalid
plans between valid ones.  R_d, bottleneck and flags bit for bit against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import oracle as O  # noqa: E402
from paper_2512_14098_amd.inputs import load_config, make_plans  # noqa: E402


@pytest.mark.parametrize("P", [1, 255, 257, 700])
@pytest.mark.parametrize("batches", [[1, 256], list(range(1, 257))])
@pytest.mark.parametrize("het,tp", [(False, False), (False, True), (True, True)])
def test_routing_shares(P, batches, het, tp):
    from paper_2512_14098_amd import cf
    print(f"coarse edges P={P} batches={len(batches)} het={het} tp={tp}", flush=True)
    cfg = load_config("c2")
    mc = dict(cfg["model"])
    if tp:
        mc["components"] = [dict(c, tp_scale={"2": 0.55, "4": 0.3, "8": 0.2}) for c in mc["components"]]
    cfg["plans"] = {"sampled": dict(cfg["plans"]["sampled"], total=P, seed=11)}
    if het:
        cfg["plans"]["sampled"]["het"] = 0.5
    tab = make_plans(cfg, cache=False)
    for f in type(tab).FIELDS:
        setattr(tab, f, getattr(tab, f).copy())
    rng = np.random.default_rng(P + len(batches))
    live = np.arange(tab.node_rep.shape[0])[:, None] < tab.n_nodes[None, :]
    tab.node_batch[...] = np.where(live, rng.choice(batches, tab.node_batch.shape), 0)
    if tp:
        tab.node_gpus[...] = np.where(live, rng.choice([1, 2, 4, 7, 8, 16], tab.node_gpus.shape), tab.node_gpus)
    if het:
        split = tab.node_rep2 > 0
        tab.node_batch2[...] = np.where(split, rng.choice(batches, split.shape), tab.node_batch2)
        tab.node_gpus2[...] = np.where(split, rng.choice([1, 2, 4], split.shape), tab.node_gpus2)
    # shares that are no tenths, a share of zero and a route that does not fit, in some plans
    two = tab.n_alt == 2
    odd = two & (rng.random(two.shape) < 0.3)
    for a in range(2):
        rows = tab.alt_w[a::2]
        rows[...] = np.where(odd, rng.integers(1, 200, two.shape), rows)
    tab.alt_w[0, ::17] = np.where(two[0, ::17], 0, tab.alt_w[0, ::17])
    tab.alt_w[1, ::17] = np.where(two[0, ::17], 10, tab.alt_w[1, ::17])
    tab.node_batch[0, 5::29] = 0
    m = O.make_model(mc)
    mom = O.trace_gen(m, [1], 2000)["moments"][0]
    desc = cf.model_desc(mc)
    md = cf.cf_trace_gen(desc, [1], 2000)[1][0].contiguous()
    rd, bn, fl = cf.cf_eval_coarse(desc, cf.DevicePlans(tab), md, 64)
    w = O.eval_coarse(m, tab, mom, 64)
    assert np.array_equal(rd.cpu().numpy().view(np.uint64), w[0].view(np.uint64))
    assert np.array_equal(bn.cpu().numpy(), w[1]) and np.array_equal(fl.cpu().numpy(), w[2])
