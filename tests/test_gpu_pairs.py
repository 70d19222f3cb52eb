"""Pair distances at the edges of their 64 x 64 tile products: spin counts
around the 4-spin words, the 32-spin steps and the sixteen waves' shares of
them, one to several replica tiles, against numpy on the same population."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 3, 4, 5, 31, 32, 33, 511, 512, 513, 545, 1027, 4099])
@pytest.mark.parametrize("R", [64, 128, 320])
def test_pair_distances_at_edges(n, R):
    from paper_2606_25203_amd import pamc
    print(f"case pair distances n={n} R={R}", flush=True)
    g = synth.csr_from_edges(n, np.arange(n - 1), np.arange(1, n), np.ones(n - 1, np.int32))
    rng = np.random.default_rng(n + R)
    base = rng.choice(np.array([-1, 1], np.int8), n)
    # copies, global flips and everything between
    flips = rng.random((R, n)) < rng.choice([0.0, 0.1, 0.5, 1.0], R)[:, None]
    s = np.where(flips, -base, base).astype(np.int8)
    inst = pamc.Instance.csr(g, replicas=R, seed=1)
    inst.set_state(s)
    i, j = np.triu_indices(R, 1)
    d = (n - (s.astype(np.int32) @ s.astype(np.int32).T)[i, j]) // 2
    d = np.minimum(d, n - d).astype(np.int64)
    mean = d.sum() / (n * len(d))
    for nbins in (1, 10, 4096):
        counts, m = inst.pair_distance_hist(nbins)
        assert np.array_equal(counts, np.bincount(np.minimum(nbins - 1, 2 * nbins * d // n), minlength=nbins))
        assert m == pytest.approx(mean, rel=1e-14, abs=0)
    # one rounding each in the division and the product: 3 units in the last place
    assert inst.pair_distance() == pytest.approx(mean, rel=1e-14, abs=0)
    inst.close()
