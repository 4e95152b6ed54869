"""cf_trace_gen at the edges of its blocks of 256 requests (one request, one short of a
block, a block, several, with and without a second seed), with every length distribution
(none, constant, lognormal, lognormal in seconds, exponential) and image rule: every trace
array and moment equals the oracle's."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import oracle as O  # noqa: E402
from tests.helpers import comp, model, rtype  # noqa: E402

MODEL = model(
    [comp("L", "LLM", [0.005, 4e-5, 0.0], x=["prompt"], decode=(0.012, 8e-5))],
    [rtype("a", ["L"], weight=3, prompt={"lognormal": [6.0, 0.5]}, out={"exp": 40.0}, images={"uniform": [0, 4]}),
     rtype("b", ["L"], weight=2, prompt={"const": 77}, out={"lognormal": [5.0, 0.6]}, images={"const": 2},
           aud_in={"lognormal_s": [1.5, 0.5]}, aud_out={"exp": 3000.0}),
     rtype("c", ["L"], weight=1)])


def _check(n, seeds):
    from paper_2512_14098_amd import cf
    tr, mom = cf.cf_trace_gen(cf.model_desc(MODEL), seeds, n)
    want = O.trace_gen(O.make_model(MODEL), seeds, n)
    got = tr.to_numpy()
    for f, _ in cf.TRACE_FIELDS:
        assert np.array_equal(got[f], want[f]), (f, n)
    assert np.array_equal(mom.cpu().numpy().view(np.uint64), want["moments"])


@pytest.mark.parametrize("n", [1, 2, 255, 256, 257, 1024, 1025, 3000])
@pytest.mark.parametrize("seeds", [[5], [6, 2 ** 63 + 1, 7]])
def test_trace_block_edges(n, seeds):
    _check(n, seeds)


@pytest.mark.parametrize("n", [(1 << 20) - 255, 1 << 20, (1 << 20) + 1, (1 << 21) + 300])
def test_block_totals_over_one_round(n):
    """4,096 block totals are scanned in one round: one round just full, the second with one
    total, the third with two."""
    print(f"trace totals: {n} requests", flush=True)
    _check(n, [5, 9])
