"""Plan enumeration where its blocks and tables change form: blocks spanning many logical plans
(small budgets, some logical plans without a plan), routing digits that wrap inside a block,
budgets that are no power of two with several GPU options, and screens whose option table does
not fit LDS.  Byte for byte against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import oracle as O  # noqa: E402
from paper_2512_14098_amd.inputs import load_config  # noqa: E402
from paper_2512_14098_amd.inputs.plans import PlanTable  # noqa: E402

EIGHT = [1, 3, 8, 16, 40, 64, 100, 256]


@pytest.mark.parametrize("name,N,batch,gpus", [
    ("c2", 3, [16], None),                      # many logical plans with few or no plans
    ("c2", 5, [16, 64], [1, 2]),
    ("c2", 13, [16, 64, 256], [1, 3]),          # a budget between powers of two
    ("c2", 12, EIGHT, [1, 2, 4, 8]),            # 160 options: the screen's work table exceeds LDS
    ("c1", 33, EIGHT, [2, 1, 8, 33]),
    ("c1", 64, [7], None),
])
def test_enumeration_edges(name, N, batch, gpus):
    from paper_2512_14098_amd import cf
    print(f"enum edges {name} N={N}", flush=True)
    mc = dict(load_config(name)["model"])
    if gpus:
        mc["components"] = [dict(c, tp_scale={"2": 0.55, "4": 0.3}) for c in mc["components"]]
    spec = {"k_s": 2, "share": True, "batch": {c["name"]: batch for c in mc["components"]}}
    if gpus:
        spec["gpus"] = {c["name"]: gpus for c in mc["components"]}
        if N < max(gpus):
            spec["gpus"] = {c["name"]: [g for g in gpus if g <= N] for c in mc["components"]}
    desc, opts = cf.model_desc(mc), cf.enum_opts(mc, spec, N)
    ldev = torch.from_numpy(cf.cf_enum_logical(desc, opts)).cuda()
    offsets, total = cf.cf_enum_count(desc, opts, ldev)
    m, oo = O.make_model(mc), O.enum_opts(mc, spec, N)
    Ls = O.enum_logical(m, oo)
    offs = np.concatenate([[0], np.cumsum([O.enum_count(m, oo, L) for L in Ls])])
    assert total == int(offs[-1])
    mom = cf.cf_trace_gen(desc, [3], 3000)[1]
    mom_h = O.trace_gen(m, [3], 3000)["moments"][0]
    mid = int(offs[len(offs) // 2])
    for first, cnt in ((0, 3001), (max(0, mid - 1500), 2049), (max(0, total - 2050), 2050), (total // 3, 1)):
        cnt = min(cnt, total - first)
        got = cf.cf_enum_plans(desc, opts, ldev, offsets, total, first, cnt).to_host()
        want = O.enum_plans(m, oo, Ls, first, cnt)
        for f in PlanTable.FIELDS:
            assert np.array_equal(getattr(got, f), getattr(want, f)), (f, first, cnt)
        rd, bn, fl = cf.cf_enum_screen(desc, opts, ldev, offsets, total, first, cnt, mom[0], N)
        w = O.eval_coarse(m, want, mom_h, N)
        assert np.array_equal(rd.cpu().numpy(), w[0]) and np.array_equal(bn.cpu().numpy(), w[1]), (first, cnt)
        assert np.array_equal(fl.cpu().numpy(), w[2]), (first, cnt)


def test_enumeration_after_a_count_finds_its_scratch():
    """cf_enum_count keeps no table but sizes the scratch for one: the enumeration that follows
    allocates no device memory (it may be under stream capture)."""
    from paper_2512_14098_amd import cf
    mc = load_config("c2")["model"]
    spec = {"k_s": 2, "share": True, "batch": {c["name"]: [16, 64] for c in mc["components"]},
            "gpus": {c["name"]: [1, 2, 4, 8] for c in mc["components"]}}
    desc, opts = cf.model_desc(mc), cf.enum_opts(mc, spec, 12)
    ldev = torch.from_numpy(cf.cf_enum_logical(desc, opts)).cuda()
    tab = cf.DevicePlans.empty(1000)
    mom = cf.cf_trace_gen(desc, [3], 100)[1]
    cf.cf_enum_screen(desc, opts, ldev, *cf.cf_enum_count(desc, opts, ldev), 0, 1000, mom[0], 12)  # code loaded
    torch.cuda.synchronize()
    cf.cf_release_scratch()
    offsets, total = cf.cf_enum_count(desc, opts, ldev)
    free = torch.cuda.mem_get_info()[0]
    cf.cf_enum_plans(desc, opts, ldev, offsets, total, 0, 1000, tab)
    torch.cuda.synchronize()
    assert torch.cuda.mem_get_info()[0] == free
    m, oo = O.make_model(mc), O.enum_opts(mc, spec, 12)
    want = O.enum_plans(m, oo, O.enum_logical(m, oo), 0, 1000)
    got = tab.to_host()
    for f in PlanTable.FIELDS:
        assert np.array_equal(getattr(got, f), getattr(want, f)), f
