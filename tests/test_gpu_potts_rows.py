"""Potts fields of a quad's rows taken together: rows that are empty, shorter
than and longer than a step's sixteen entries, in every order within a quad,
classes that end inside a quad, packed and plain label sums, against the
oracle."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


def from_edges(n, edges, c):
    u, v = np.array(edges).T
    return synth.csr_from_edges(n, u, v, np.full(len(u), c, np.int32))


def star(n, leaves):
    return [(0, n - 1 - i) for i in range(leaves)] + [(i, i + 1) for i in range(2, 9)]


GRAPHS = {
    "isolated": lambda c: from_edges(61, [(3, 58), (4, 30), (17, 18), (30, 31)], c),  # most rows empty
    "star": lambda c: from_edges(75, star(75, 60), c),                                # one long row
    "complete": lambda c: from_edges(23, [(i, j) for i in range(23) for j in range(i)], c),  # a class per vertex
    "bipartite": lambda c: from_edges(50, [(i, j) for i in range(17) for j in range(17, 50) if (i * j) % 3], c),
}


@pytest.mark.parametrize("gname", list(GRAPHS))
@pytest.mark.parametrize("K,rule", [(2, 0), (3, 0), (3, 1), (4, 0)])
@pytest.mark.parametrize("c", [1, 4000])  # packed label sums, and fields beyond them for K > 2
def test_potts_rows_of_a_quad(gname, K, rule, c):
    from paper_2606_25203_amd import pamc
    g = GRAPHS[gname](c)
    print(f"case potts rows {gname} K={K} rule={rule} c={c}", flush=True)
    inst = pamc.Instance.potts(g, K, replicas=192, seed=7, potts_rule=rule, gamma=1.0)
    o = oracle.Oracle.potts(g.n, g.row_ptr, g.col, g.w, K, 192, 7, rule=rule, gamma=1.0)
    for beta, sweeps in ((0.3 / c, 2), (1.1 / c, 3)):
        inst.sweep(beta, sweeps)
        o.sweep(beta, sweeps)
        for name, a, b in zip(("labels", "fields", "energies", "family"), inst.state(), o.state()):
            if name != "fields":
                assert np.array_equal(a, b), f"{gname} K={K} rule={rule} c={c} beta={beta}: {name} differ"
    inst.close()
