"""Matrix-core fields in 16-replica work-groups at their edges: vertex counts
around the 4, 16 and 64 of quads, row tiles and columns, classes of more row
tiles than waves, of one vertex, ending inside a quad, one class after itself
(sweep boundaries), both rules, against the oracle."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


def edges(n, pairs, seed):
    u, v = np.array(pairs, np.int64).T
    w = np.random.default_rng(seed).choice(np.array([-1, 1, 2], np.int32), len(u))
    return synth.csr_from_edges(n, u, v, w)


def complete(n):
    return edges(n, [(i, j) for i in range(n) for j in range(i)], n)


def blocks(sizes, per, seed):
    """Classes of the given sizes: `per` edges from each vertex to every other class."""
    rng = np.random.default_rng(seed)
    start = np.concatenate([[0], np.cumsum(sizes)])
    pairs = set()
    for a in range(len(sizes)):
        for b in range(a):
            for u in range(start[a], start[a + 1]):
                for v in rng.choice(np.arange(start[b], start[b + 1]), min(per, sizes[b]), replace=False):
                    pairs.add((u, int(v)))
    return edges(int(start[-1]), sorted(pairs), seed)


CASES = {
    "two": lambda: complete(2),
    "complete17": lambda: complete(17),
    "complete63": lambda: complete(63),
    "complete65": lambda: complete(65),
    "bipartite300": lambda: blocks([150, 150], 40, 1),
    "bipartite1024": lambda: blocks([512, 512], 60, 2),  # 32 row tiles to a class
    "uneven": lambda: blocks([1, 130, 3, 67, 18, 200], 60, 3),
    "n129": lambda: synth.random_graph(129, 1500, 4, weights="pm1"),
    "n1023": lambda: synth.random_graph(1023, 40000, 5),
}


@pytest.mark.parametrize("gname", list(CASES))
@pytest.mark.parametrize("rule", [0, 1])
def test_groups_at_edges(monkeypatch, gname, rule):
    from paper_2606_25203_amd import pamc
    monkeypatch.setenv("PAMC_TILE", "2")
    g = CASES[gname]()
    for R in (64, 192):
        print(f"case mfma groups {gname} rule={rule} R={R}", flush=True)
        inst = pamc.Instance.csr(g, replicas=R, seed=3, rule=rule)
        o = oracle.Oracle.sparse(g.n, g.row_ptr, g.col, g.w, R, 3, rule=rule)
        for beta, k in ((0.0, 1), (0.1, 7), (0.8, 4)):
            inst.sweep(beta, k)
            o.sweep(beta, k)
            for name, a, b in zip(("spins", "fields", "energies", "family"), inst.state(), o.state()):
                assert np.array_equal(a, b), f"{gname} rule={rule} R={R} beta={beta}: {name} differ"
        inst.close()
