"""Bit-packed sweeps (couplings of one magnitude): states, energies and runs
against the oracle, over every tile-group and vertex grouping, both update
rules, couplings of one sign, of the other and of both, rows up to the longest
taken, and populations whose tile count no group divides."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pamc():
    from paper_2606_25203_amd import pamc as p
    return p


def scaled(g, c):
    return synth.Graph(g.n, g.row_ptr, g.col, (g.w * c).astype(np.int32))


def star(n, leaves):
    """A path over n vertices with vertex 0 also joined to the last `leaves`."""
    u = list(range(n - 1)) + [0] * leaves
    v = list(range(1, n)) + list(range(n - leaves, n))
    return synth.csr_from_edges(n, np.array(u), np.array(v), np.ones(len(u), np.int32))


GRAPHS = {
    "even_torus": lambda: synth.torus(14, 10, 2),
    "odd_torus": lambda: synth.torus(9, 7, 3),                    # three or more classes, ragged quads
    "unit": lambda: synth.random_graph(203, 1400, 17),            # J = -1 everywhere
    "minus": lambda: scaled(synth.random_graph(101, 300, 4), -3),  # J = +3 everywhere
    "both": lambda: scaled(synth.random_graph(157, 800, 6, weights="pm1"), 1000),
    "isolated": lambda: synth.random_graph(61, 20, 9),            # vertices without neighbours
    "long_row": lambda: star(300, 254),                           # 256 entries, the most taken
    "two": lambda: synth.csr_from_edges(2, np.array([0]), np.array([1]), np.array([5])),
}


def same_state(inst, o, what):
    for name, a, b in zip(("spins", "fields", "energies", "family"), inst.state(), o.state()):
        assert np.array_equal(a, b), f"{what}: {name} differ"


@pytest.mark.parametrize("form", [0, 1, 2, 3, 4, 5])
@pytest.mark.parametrize("rule", [0, 1])
@pytest.mark.parametrize("gname", list(GRAPHS))
def test_bit_sweeps_match_oracle(pamc, monkeypatch, form, rule, gname):
    monkeypatch.setenv("PAMC_BITS", "1")
    monkeypatch.setenv("PAMC_BITS_FORM", str(form))
    monkeypatch.setenv("PAMC_BITS_QPW", "2" if form % 2 else "1")
    g = GRAPHS[gname]()
    c = int(np.abs(g.w).max())
    for R, seed in ((64, 1), (192, 2), (512, 3)):  # 1, 3 and 8 tiles
        print(f"case bits {gname} form={form} rule={rule} R={R}", flush=True)
        inst = pamc.Instance.csr(g, replicas=R, seed=seed, rule=rule)
        o = oracle.Oracle.sparse(g.n, g.row_ptr, g.col, g.w, R, seed, rule=rule)
        for beta, k in [(0.01, 1), (0.3, 3), (1.2, 2), (0.0, 1), (-0.4, 1)]:
            inst.sweep(beta / c, k)
            o.sweep(beta / c, k)
            same_state(inst, o, f"beta={beta}")
        kw = dict(beta0=0.1 / c, dbeta=0.1 / c, steps=30, sweeps=2, augmented=1, z_rst=20, n_top=5, mis_trials=3,
                  win_short=4, win_long=6, max_distinct_short=2, max_distinct_long=3, tau=3)
        res = inst.anneal(pamc.schedule(**kw))
        ores = o.anneal(oracle.default_schedule(**kw))
        for f in ("best_cut", "best_energy", "steps_run", "n_cluster_moves", "n_reheats", "n_reversals", "n_restarts"):
            assert getattr(res, f) == getattr(ores, f), f
        same_state(inst, o, "run")
        inst.close()


def test_bit_batch_of_uneven_instances(pamc, monkeypatch):
    """Bit-packed instances of uneven class counts, sizes and tile counts in
    one batch with instances of other forms, and through the entry point that
    allocates nothing: each as in its own run."""
    graphs = [synth.torus(40, 60, 1), synth.random_graph(2500, 30000, 2), synth.torus(45, 51, 3),
              synth.random_graph(2100, 4000, 4, weights="pm1"), scaled(synth.torus(12, 9, 5), 200),
              synth.random_graph(301, 2500, 3)]
    reps = [128, 256, 192, 64, 128, 256]
    sched = [pamc.schedule(beta0=0.1, dbeta=0.1, steps=12 + i, sweeps=1 + i % 3, augmented=1, z_rst=10, n_top=4, tau=3)
             for i in range(len(graphs))]
    alone = []
    for g, R, s in zip(graphs, reps, sched):
        inst = pamc.Instance.csr(g, replicas=R, seed=R)
        r = inst.anneal(s)
        alone.append((r.best_cut, r.sum_lnq, inst.state(), inst.best()[2]))
        inst.close()
    for entry in (pamc.anneal_batch, pamc.anneal_batch_noalloc):
        print("case bit-packed batch", entry.__name__, flush=True)
        insts = [pamc.Instance.csr(g, replicas=R, seed=R) for g, R in zip(graphs, reps)]
        for inst, r, want in zip(insts, entry(insts, sched), alone):
            assert (r.best_cut, r.sum_lnq) == want[:2]
            assert all(np.array_equal(a, b) for a, b in zip(inst.state(), want[2]))
            assert np.array_equal(inst.best()[2], want[3])
            inst.close()
