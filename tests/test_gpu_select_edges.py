"""cf_select_topk at the edges of its radix select: ties in R_d, one value everywhere, keys
that differ in their lowest or highest bits only, k below, at and above the kept count,
sizes around the four plans of a thread, and a flags array that is not word-aligned.
Expected: numpy's lexsort by (R_d bits descending, id ascending)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _values(kind, P, rng):
    if kind == "mixed":
        return rng.lognormal(1.0, 2.0, P)
    if kind == "ties":
        return rng.integers(1, 5, P).astype(np.float64)
    if kind == "equal":
        return np.full(P, 3.25)
    if kind == "low":  # neighbours of 1.0
        return (np.float64(1.0).view(np.int64) + rng.integers(0, 3, P)).view(np.float64)
    return np.where(rng.random(P) < 0.5, 0.0, np.inf)  # "far": the widest range of bits


@pytest.mark.parametrize("kind", ["mixed", "ties", "equal", "low", "far"])
@pytest.mark.parametrize("P,k", [(1, 1), (3, 2), (5, 5), (1023, 100), (1025, 2000), (70001, 997), (70001, 65536)])
def test_topk_edges(kind, P, k):
    from paper_2512_14098_amd import cf
    rng = np.random.default_rng(P * 7 + k)
    rd = _values(kind, P, rng)
    flags = rng.integers(0, 16, P + 1).astype(np.uint8)
    dev = torch.from_numpy(flags).cuda()
    for off in (0, 1):  # off = 1: the flags start at an odd address
        f = dev[off:off + P]
        got = cf.cf_select_topk(torch.from_numpy(rd).cuda(), f, k).cpu().numpy()
        kept = np.nonzero(flags[off:off + P] & 1)[0]
        bits = rd.view(np.uint64)[kept]
        want = kept[np.lexsort((kept, ~bits))][:k]
        assert np.array_equal(got, want), (kind, P, k, off)
