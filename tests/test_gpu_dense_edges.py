"""Dense instances at the edges of their tiles: vertex counts around the
64-spin blocks, the 128-column stages and the 1,024-row super-blocks, replica
counts of each field-product tile (64, 128, 256, ragged and several), narrow
and wide couplings, both rules, and thresholds that rise (a negative beta),
against the oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pamc():
    from paper_2606_25203_amd import pamc as p
    return p


def couplings(n, lim, seed):
    J = np.triu(np.random.default_rng(seed).integers(-lim, lim + 1, size=(n, n)), 1).astype(np.int8)
    return (J + J.T).astype(np.int8)


def same_state(inst, o, what):
    for name, a, b in zip(("spins", "fields", "energies", "family"), inst.state(), o.state()):
        assert np.array_equal(a, b), f"{what}: {name} differ"


SIZES = ([(n, R) for n in (1, 2, 63, 65, 129, 1025) for R in (64, 128, 192, 320, 512)]
         + [(n, R) for n in (1023, 1024, 1089, 2049) for R in (64, 192, 320)])


@pytest.mark.parametrize("n,R", SIZES)
def test_dense_edges(pamc, n, R):
    big = n > 1000
    rule = (n + R // 64) % 2
    for lim in (1, 127):
        J = couplings(n, lim, 7 * n + R)
        print(f"case dense edges n={n} R={R} rule={rule} lim={lim}", flush=True)
        inst = pamc.Instance.dense(J, replicas=R, seed=n + R, rule=rule)
        o = oracle.Oracle.dense(J, R, n + R, rule=rule)
        scale = 1.0 / (lim * np.sqrt(n))
        for beta, k in ((0.0, 1), (0.7 * scale, 1 if big else 3), (-0.5 * scale, 1), (2.0 * scale, 1)):
            inst.sweep(beta, k)
            o.sweep(beta, k)
            same_state(inst, o, f"n={n} R={R} rule={rule} lim={lim} beta={beta}")
        inst.close()


@pytest.mark.parametrize("rule", [0, 1])
def test_dense_table_beyond_lds(pamc, rule):
    """A threshold table wider than the part of it that a work-group keeps in
    LDS, and replicas that resampling has moved between the buffers."""
    n, R = 1100, 128
    J = couplings(n, 127, 3)
    print(f"case dense wide table rule={rule}", flush=True)
    inst = pamc.Instance.dense(J, replicas=R, seed=6, rule=rule)
    o = oracle.Oracle.dense(J, R, 6, rule=rule)
    assert 2 * o.X + 1 > 4 * 32768
    for beta in (1e-5, 3e-4, 2e-3):
        inst.sweep(beta, 1)
        o.sweep(beta, 1)
        inst.resample(1e-5)
        o.resample(1e-5)
        same_state(inst, o, f"rule={rule} beta={beta}")
    inst.close()
