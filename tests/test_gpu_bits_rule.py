"""The choice between bit-packed and other sweeps by the sweeps of a step: one
instance called with few and many sweeps in turn (which changes its launches),
runs of one and of several sweeps per step, and a batch of both, against the
oracle; class orders longer than the part shuffled at a time."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

GRAPHS = {
    "tile": lambda: synth.random_graph(150, 500, 3, weights="pm1"),     # a work-group per tile for few sweeps
    "pull": lambda: synth.random_graph(2600, 7000, 4, weights="pm1"),   # per-class launches for few
    "torus": lambda: synth.torus(50, 48, 5),
}


def same_state(inst, o, what):
    for name, a, b in zip(("spins", "fields", "energies", "family"), inst.state(), o.state()):
        assert np.array_equal(a, b), f"{what}: {name} differ"


@pytest.mark.parametrize("gname", list(GRAPHS))
@pytest.mark.parametrize("rule", [0, 1])
def test_sweep_counts_in_turn(gname, rule):
    from paper_2606_25203_amd import pamc
    g = GRAPHS[gname]()
    inst = pamc.Instance.csr(g, replicas=128, seed=5, rule=rule)
    o = oracle.Oracle.sparse(g.n, g.row_ptr, g.col, g.w, 128, 5, rule=rule)
    for i, k in enumerate((1, 1, 1, 1, 6, 6, 6, 6, 1, 6, 30, 1, 2, 3, 4, 5)):
        print(f"case sweep counts {gname} rule={rule} call {i}: {k} sweeps", flush=True)
        inst.sweep(0.1 + 0.05 * i, k)
        o.sweep(0.1 + 0.05 * i, k)
        same_state(inst, o, f"{gname} rule={rule} call {i}")
    for sweeps in (1, 6, 2):
        kw = dict(beta0=0.2, dbeta=0.1, steps=6, sweeps=sweeps)
        assert inst.anneal(pamc.schedule(**kw)).best_cut == o.anneal(oracle.default_schedule(**kw)).best_cut
        same_state(inst, o, f"{gname} rule={rule} run of {sweeps}")
    inst.close()


@pytest.mark.parametrize("sweeps", [(1, 1, 1), (1, 5, 2)])
def test_batch_of_both(sweeps):
    from paper_2606_25203_amd import pamc
    print(f"case batch sweeps={sweeps}", flush=True)
    gs = [make() for make in GRAPHS.values()]
    insts = [pamc.Instance.csr(g, replicas=64, seed=9 + i) for i, g in enumerate(gs)]
    kws = [dict(beta0=0.2, dbeta=0.1, steps=5, sweeps=s) for s in sweeps]
    pamc.anneal_batch(insts, [pamc.schedule(**kw) for kw in kws])
    for i, (g, inst, kw) in enumerate(zip(gs, insts, kws)):
        o = oracle.Oracle.sparse(g.n, g.row_ptr, g.col, g.w, 64, 9 + i)
        o.anneal(oracle.default_schedule(**kw))
        same_state(inst, o, f"batch {i} of {sweeps}")
        inst.close()


def test_many_classes_shuffled():
    """A complete graph: a class per vertex, so 9 sweeps' orders (2,340
    entries) exceed the part that is shuffled at a time."""
    from paper_2606_25203_amd import pamc
    n = 260
    u, v = np.triu_indices(n, 1)
    g = synth.csr_from_edges(n, u, v, np.random.default_rng(1).integers(1, 3, len(u)).astype(np.int32))
    print("case many classes", flush=True)
    inst = pamc.Instance.csr(g, replicas=64, seed=2)
    o = oracle.Oracle.sparse(g.n, g.row_ptr, g.col, g.w, 64, 2)
    inst.sweep(0.02, 9)
    o.sweep(0.02, 9)
    same_state(inst, o, "many classes")
    inst.close()
