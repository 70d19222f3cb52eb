"""Which sweep form an instance takes, seen from outside: the sweep launches
that the library's own counter reports (one for a step of a matrix-core or
gathered tile form, one per colour class and sweep for the others), with
results as in the other forms."""
import numpy as np
import pytest

import oracle
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


@pytest.mark.parametrize("gname", ["tile", "pull", "torus"])
def test_sweep_counts_change_no_launch_state(pamc, gname):
    """Sweep calls of few and of many sweeps, each in its own form, leave what
    the others' launches use in place: a captured sequence of both can be
    replayed after (and between) eager calls of either, and takes no wait
    while it is captured."""
    import torch
    g = {"tile": lambda: synth.random_graph(150, 500, 3, weights="pm1"),
         "pull": lambda: synth.random_graph(2600, 7000, 4, weights="pm1"),
         "torus": lambda: synth.torus(50, 48, 5)}[gname]()
    stream = torch.cuda.Stream()
    inst = pamc.Instance.csr(g, replicas=128, seed=5, stream=stream.cuda_stream)
    o = oracle.Oracle.sparse(g.n, g.row_ptr, g.col, g.w, 128, 5)

    def eager(betas):
        for beta, k in betas:
            inst.sweep(beta, k)
            o.sweep(beta, k)

    def same(what):
        for name, a, b in zip(("spins", "fields", "energies", "family"), inst.state(), o.state()):
            assert np.array_equal(a, b), f"{what}: {name} differ"

    print("case captured sweeps", gname, flush=True)
    eager([(0.2, 6)])
    same("before")
    captured = [(0.3, 1), (0.35, 1), (0.4, 1), (0.45, 1), (0.5, 7), (0.5, 7), (0.55, 7), (0.6, 1)]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        for beta, k in captured:
            inst.sweep(beta, k)
    for rep in range(4):
        with torch.cuda.stream(stream):
            graph.replay()
        for beta, k in captured:
            o.sweep(beta, k)
        same(f"replay {rep}")
        eager([(0.3, 1)] * 4 if rep % 2 else [(0.3, 6)] * 4)
        same(f"after replay {rep}")
    inst.close()


def launches_of(pamc, inst, k):
    pamc.pamc_profile_enable(inst.h, True)
    inst.sweep(0.5, k)
    n = pamc.pamc_profile_read(inst.h)["launches"]
    pamc.pamc_profile_enable(inst.h, False)
    return n


@pytest.mark.parametrize("sweeps", [1, 40])
def test_tuning_at_some_sweeps_keeps_the_choice_for_others(pamc, monkeypatch, sweeps):
    """A small graph whose step of one sweep is one launch and whose steps of
    many go bit-packed: tuned at either count, it still takes its form at the
    other, a new instance of the shape does too, and one made under PAMC_BITS=1
    goes bit-packed always."""
    g = synth.random_graph(600 + sweeps, 2100, 3)  # a shape of its own: tuned shapes are remembered
    make = lambda seed: pamc.Instance.csr(g, replicas=256, seed=seed)
    inst = make(1)
    ncls = inst.info().num_classes
    print(f"case tuned at {sweeps}, {ncls} classes", flush=True)
    other = 41 - sweeps
    form = {1: 1, 40: 40 * ncls}
    assert [launches_of(pamc, inst, k) for k in (1, 40)] == [form[1], form[40]]
    before = inst.state()
    t = inst.autotune(0.5, sweeps=sweeps, force=True)
    assert t.candidates > 2 and t.best_ms_per_sweep <= t.default_ms_per_sweep
    assert all(np.array_equal(a, b) for a, b in zip(before, inst.state()))
    new = make(2)
    for i in (inst, new):
        assert launches_of(pamc, i, other) == form[other]
    assert new.autotune(0.5, sweeps=other).cached == 1
    assert launches_of(pamc, new, other) == form[other]
    monkeypatch.setenv("PAMC_BITS", "1")
    forced = make(3)
    assert launches_of(pamc, forced, 1) == ncls
    for i in (inst, new, forced):
        i.close()


def long_rows(n, rows, length, seed):
    """A ring with `rows` vertices of about `length` neighbours, weights 1."""
    rng = np.random.default_rng(seed)
    pairs = {(i, i + 1) for i in range(rows, n - 1)}
    for k in range(rows):
        pairs |= {(k, int(v)) for v in rng.choice(np.arange(rows, n), length, replace=False)}
    u, v = np.array(sorted(pairs)).T
    return synth.csr_from_edges(n, u, v, np.ones(len(u), np.int32))


@pytest.mark.parametrize("n,rows,R,pull,hubs", [
    (2600, 4, 64, 0, 0),       # incremental fields, as for other magnitudes
    (2600, 1, 64, 0, 1),       # both field forms
    (2600, 4, 512, 1, 0),      # gathered
    (1500, 4, 64, 1, 0),       # a work-group per tile
])
def test_rows_far_longer_than_the_others(pamc, n, rows, R, pull, hubs):
    """Graphs of one magnitude with a few rows of more than 128 entries: the
    field form they take, and their states in it."""
    g = long_rows(n, rows, 200, n + rows)
    print(f"case long rows n={n} rows={rows} R={R}", flush=True)
    inst = pamc.Instance.csr(g, replicas=R, seed=3)
    info = inst.info()
    assert (info.pull, info.hubs) == (pull, hubs)
    o = oracle.Oracle.sparse(g.n, g.row_ptr, g.col, g.w, R, 3)
    for beta, k in ((0.2, 1), (0.6, 4), (1.5, 2)):
        inst.sweep(beta, k)
        o.sweep(beta, k)
    kw = dict(beta0=0.2, dbeta=0.1, steps=8, sweeps=3)
    assert inst.anneal(pamc.schedule(**kw)).best_cut == o.anneal(oracle.default_schedule(**kw)).best_cut
    for name, a, b in zip(("spins", "fields", "energies", "family"), inst.state(), o.state()):
        assert np.array_equal(a, b), name
    inst.close()


def test_reported_form_is_the_one_launched(pamc, monkeypatch):
    """bit_sweeps tells from how many sweeps on a step of a small graph is no
    longer one launch; graphs that never pack report 0."""
    g = synth.random_graph(620, 2170, 3)
    inst = pamc.Instance.csr(g, replicas=256, seed=1)
    info = inst.info()
    print("case reported form", info.bit_sweeps, info.bit_tiles, flush=True)
    assert 1 < info.bit_sweeps < 40 and info.bit_tiles != 0 and info.tile_sweeps == 1
    for k in (info.bit_sweeps - 1, info.bit_sweeps):
        assert launches_of(pamc, inst, k) == (k * info.num_classes if k >= info.bit_sweeps else 1)
    inst.close()
    others = [pamc.Instance.csr(synth.random_graph(300, 2400, 5), replicas=128, seed=1),     # matrix-core tiles
              pamc.Instance.csr(synth.torus(50, 48, 5), replicas=128, seed=1, fields="push"),
              pamc.Instance.potts(synth.random_graph(300, 600, 1), 3, replicas=64, seed=1),
              pamc.Instance.dense_random(100, 1, replicas=64, seed=1)]
    monkeypatch.setenv("PAMC_BITS", "0")
    others.append(pamc.Instance.csr(g, replicas=256, seed=1))
    assert [(i.info().bit_sweeps, i.info().bit_tiles) for i in others] == [(0, 0)] * 5
    monkeypatch.setenv("PAMC_BITS", "1")
    forced = pamc.Instance.csr(synth.torus(100, 200, 1), replicas=4096, seed=1)
    assert (forced.info().bit_sweeps, forced.info().bit_tiles) == (1, 4)
    for i in others + [forced]:
        i.close()
