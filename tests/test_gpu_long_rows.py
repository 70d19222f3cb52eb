"""Fields of rows around the length from which four waves share one, recomputed
from the population (creation, loaded spins, the snapshot), and their updates
by scattered flips, against numpy and the oracle."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


def hubs(lengths, n, seed):
    """Vertex k joined to lengths[k] others, on a ring."""
    rng = np.random.default_rng(seed)
    pairs = {(i, (i + 1) % n) for i in range(len(lengths), n - 1)}
    for k, m in enumerate(lengths):
        pairs |= {(k, int(v)) for v in rng.choice(np.arange(len(lengths), n), m, replace=False)}
    u, v = np.array(sorted(pairs)).T
    return synth.csr_from_edges(n, u, v, rng.integers(-5, 6, len(u)).astype(np.int32) * 2 + 1)


@pytest.mark.parametrize("lengths", [(510, 511), (512, 513), (1023, 900), (1400,), (515, 600, 700, 512)])
@pytest.mark.parametrize("flags", ["default", "push", "pull"])
def test_long_rows(lengths, flags):
    from paper_2606_25203_amd import pamc
    n, R = 1500, 192
    print(f"case long rows {lengths} {flags}", flush=True)
    g = hubs(lengths, n, sum(lengths))
    kw = {} if flags == "default" else {"fields": flags}
    inst = pamc.Instance.csr(g, replicas=R, seed=4, **kw)
    o = oracle.Oracle.sparse(g.n, g.row_ptr, g.col, g.w, R, 4)

    def same(what):
        for name, a, b in zip(("spins", "fields", "energies", "family"), inst.state(), o.state()):
            assert np.array_equal(a, b), f"{lengths} {flags} {what}: {name} differ"

    same("creation")
    for beta, k in ((0.02, 2), (0.3, 3)):
        inst.sweep(beta, k)
        o.sweep(beta, k)
        same(f"beta={beta}")
    s = np.random.default_rng(1).choice(np.array([-1, 1], np.int8), (R, n))
    inst.set_state(s)
    got, h, E, _ = inst.state()
    J = np.zeros((n, n), np.int64)
    for v in range(n):
        J[v, g.col[g.row_ptr[v]:g.row_ptr[v + 1]]] = g.w[g.row_ptr[v]:g.row_ptr[v + 1]]
    want = -(s.astype(np.int64) @ J)  # J_ij = -w_ij
    assert np.array_equal(got, s) and np.array_equal(h, want)
    assert np.array_equal(E, -(s * want).sum(axis=1) // 2)
    inst.close()
