"""Which sweep form an instance takes, seen from outside: the sweep launches
that the library's own counter reports (one for a step of a matrix-core or
gathered tile form, one per colour class and sweep for the others), with
results as in the other forms."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pamc():
    from paper_2606_25203_amd import pamc as p
    return p


@pytest.mark.parametrize("weights", ["unit", "two"])
@pytest.mark.parametrize("count", [30, 33, 130])
def test_matrix_core_batch_is_one_launch_a_step(pamc, weights, count):
    """Batches of matrix-core tile instances keep that form whatever their
    size: work-groups of 16 replicas (120 tiles), of a tile with 16 waves (132)
    and with 8 (520); couplings of one magnitude too."""
    g = synth.random_graph(301, 2500, 3)
    if weights == "two":
        g = synth.Graph(g.n, g.row_ptr, g.col, g.w.copy())
        src = np.repeat(np.arange(g.n), np.diff(g.row_ptr))
        g.w[(src + g.col) % 2 == 0] = 2
    steps, sweeps = 6, 2
    sched = pamc.schedule(beta0=0.1, dbeta=0.1, steps=steps, sweeps=sweeps)
    print(f"case batch of {count} matrix-core tile instances, {weights}", flush=True)
    insts = [pamc.Instance.csr(g, replicas=256, seed=100 + k) for k in range(count)]
    assert insts[0].info().tile_sweeps == 2
    pamc.pamc_profile_enable(insts[0].h, True)
    res = pamc.anneal_batch(insts, [sched] * count)
    assert pamc.pamc_profile_read(insts[0].h)["launches"] == steps
    for k in range(0, count, 7 if count < 100 else 31):
        alone = pamc.Instance.csr(g, replicas=256, seed=100 + k)
        r = alone.anneal(sched)
        assert (r.best_cut, r.sum_lnq) == (res[k].best_cut, res[k].sum_lnq), k
        for a, b in zip(alone.state(), insts[k].state()):
            assert np.array_equal(a, b), k
        alone.close()
    for i in insts:
        i.close()
