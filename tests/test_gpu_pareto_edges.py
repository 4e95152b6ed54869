"""cf_pareto at the edges of its blocks of 256 rows and slices of survivors, for every row
length: rows with ties, duplicates, zeros, negative and infinite entries; keep flags and
the flags of the pruned plans equal the oracle's all-pairs definition."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import oracle as O  # noqa: E402


@pytest.mark.parametrize("T", [1, 2, 3, 4, 5, 8])
@pytest.mark.parametrize("n", [1, 3, 255, 256, 257, 1500, 9001])
def test_pareto_edges(T, n):
    from paper_2512_14098_amd import cf
    rng = np.random.default_rng(100 * T + n)
    g = rng.integers(-2, 6 if n < 300 else 40, (n, T)).astype(np.float64)
    if T > 2:  # an anti-correlated column keeps many rows undominated
        g[:, 0] = 40.0 - g[:, 1] - 0.5 * g[:, 2]
    g[rng.random(n) < 0.02] = np.inf
    g[rng.random(n) < 0.05] = g[0]
    ids = rng.permutation(2 * n)[:n].astype(np.int32)
    flags = torch.full((2 * n,), 9, dtype=torch.uint8, device="cuda")
    keep = cf.cf_pareto(torch.from_numpy(g).cuda(), torch.from_numpy(ids).cuda(), flags).cpu().numpy()
    want = np.asarray(O.pareto(g)).astype(np.uint8)
    assert np.array_equal(keep, want)
    wf = np.full(2 * n, 9, np.uint8)
    wf[ids[want == 0]] = 8
    assert np.array_equal(flags.cpu().numpy(), wf)
