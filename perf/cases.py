"""The work that the library's speed is judged by.

Twelve listed cases, and `draw` for more of the same ranges: annealing runs
of one instance of each kind (sparse Max-Cut graphs from a few hundred
vertices to the 20,000 of the largest torus, Max-3-Cut as a one-hot embedding
and as Potts labels, dense couplings up to n = 100,000), a loop that a
program writes itself from the primitives, a batch of uneven small instances,
a burst of served requests, and the population's diversity histogram.  Sizes
are those of the benchmark workloads and of the request stream, shortened in
beta steps so that a pass stays below a second, beside odd and ragged ones.

A pass re-draws the population from its seed and runs to the end, so that it
can be repeated on the same state and gives the same outputs: the best cut,
its energy and configuration, the run's trace, and the energy and ancestor of
every replica at its end.
"""
import math
from types import SimpleNamespace

import numpy as np

from paper_2606_25203_amd import pamc

RULES = {"heatbath": pamc.HEATBATH, "metropolis": pamc.METROPOLIS}


def listed():
    return [
        # the smallest run anybody makes: a first try or a unit test of a
        # program; launches and waits count, and the whole population is read
        dict(name="gnm300_first_try", family="gnm", n=300, m=2400, weights="one", R=128, steps=20, sweeps=3,
             beta0=0.1, beta1=3.0, rule="heatbath", augmented=False, snapshot=True),
        # the G1-shaped benchmark run: one dense-ish instance of 800 vertices
        dict(name="gnm800_plain", family="gnm", n=800, m=19176, weights="one", R=256, steps=50, sweeps=5,
             beta0=0.1, beta1=3.0, rule="heatbath", augmented=False, snapshot=False),
        # the headline run (G81 shape), its first 120 of 500 beta steps, with
        # stagnation control and cluster moves
        dict(name="torus100x200_augmented", family="torus", width=100, height=200, R=4096, steps=120, sweeps=10,
             beta0=0.1, beta1=2.48, rule="heatbath", augmented=True, n_top=128, snapshot=False),
        # a program's own loop over the primitives, ln Q read at every
        # resampling, on a sparse graph of odd size with +-1 weights
        dict(name="gnm5003_own_loop", family="loop", n=5003, m=22510, weights="pm1", R=512, steps=60, sweeps=5,
             beta0=0.1, beta1=2.5, rule="metropolis"),
        # the heavier half of the request stream: a graph of average degree 34
        dict(name="gnm11999_degree34", family="gnm", n=11999, m=203983, weights="one", R=512, steps=60, sweeps=5,
             beta0=0.1, beta1=2.5, rule="heatbath", augmented=False, snapshot=False),
        # Max-3-Cut through the one-hot embedding (a hub of 21,000 neighbours)
        dict(name="max3cut7000_embedding", family="max3cut", n=7000, m=21000, R=2048, steps=60, sweeps=10,
             beta0=0.1, beta1=1.3, rule="heatbath", augmented=True, n_top=64),
        # the same graph with 3-state Potts labels
        dict(name="potts7000_softmax", family="potts", n=7000, m=21000, K=3, potts_rule=pamc.POTTS_SOFTMAX, gamma=1.0,
             R=2048, steps=40, sweeps=10, beta0=0.1, beta1=1.7, augmented=True, n_top=64),
        # the fully connected +-1 instance of the scalability experiment
        dict(name="dense100000", family="dense_random", n=100000, R=256, steps=12, sweeps=1, scale0=0.1, scale1=3.0,
             rule="heatbath"),
        # an uploaded dense int8 matrix of ragged size, smallest population
        dict(name="dense2047_int8", family="dense_i8", n=2047, jmax=100, R=64, steps=30, sweeps=2, scale0=0.1,
             scale1=3.0, rule="metropolis"),
        # many small instances of uneven size in one batched run
        dict(name="batch48_mixed", family="batch", count=48, n_min=200, n_max=2000, R=256, steps=40, sweeps=5,
             beta0=0.1, beta1=3.0),
        # a burst of requests to the continuous-batching server, host
        # preparation included (the request stream's sizes and degrees)
        dict(name="served32_burst", family="served", count=32, n_min=800, n_max=20000, R=512, steps=40, sweeps=5,
             beta0=0.1, beta1=3.0),
        # the diversity diagnostic over all pairs of a large population
        dict(name="diversity20000_R1024", family="diversity", width=100, height=200, R=1024, nbins=64),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _odd(rng, v):
    return v + 1 if v % 2 == 0 and rng.random() < 0.5 else v


def draw(rng):
    family = rng.choice(["gnm", "gnm", "torus", "torus", "loop", "max3cut", "potts", "dense_random", "dense_i8", "batch",
                         "served", "diversity"])
    rule = rng.choice(["heatbath", "heatbath", "metropolis"])
    R = 64 * _log_int(rng, 1, 64)
    # steps for a budget of visits, so that no drawn run is longer than the
    # listed ones
    def steps(n, sweeps, budget):
        return max(8, min(120, int(budget / (n * R * sweeps))))

    if family in ("gnm", "loop"):
        n = _odd(rng, _log_int(rng, 200, 20000))
        R = min(R, 1024)
        m = min(int(n * rng.uniform(4.0, 50.0) / 2), n * (n - 1) // 2)
        weights = rng.choice(["one", "pm1", "wide"])
        sweeps = rng.randint(1, 10)
        case = dict(family=family, n=n, m=m, weights=weights, R=R, steps=min(60, steps(n, sweeps, 2e9)), sweeps=sweeps,
                    beta0=0.1, beta1=rng.uniform(1.0, 4.0), rule=rule)
        if family == "gnm":
            case.update(augmented=rng.random() < 0.4, n_top=max(1, R // 32), snapshot=n * R < 300000)
        return case
    if family == "torus":
        w, h = _odd(rng, _log_int(rng, 8, 140)), _odd(rng, _log_int(rng, 8, 140))
        sweeps = rng.randint(2, 10)
        return dict(family=family, width=w, height=h, R=R, steps=steps(w * h, sweeps, 5e10), sweeps=sweeps, beta0=0.1,
                    beta1=rng.uniform(1.0, 5.0), rule=rule, augmented=rng.random() < 0.7, n_top=max(1, R // 32),
                    snapshot=w * h * R < 300000)
    if family in ("max3cut", "potts"):
        n = _odd(rng, _log_int(rng, 300, 7000))
        m = int(n * rng.uniform(2.0, 8.0) / 2)
        R = min(R, 2048)
        sweeps = rng.randint(2, 10)
        case = dict(family=family, n=n, m=m, R=R, steps=min(60, steps(3 * n, sweeps, 1.2e10)), sweeps=sweeps, beta0=0.1,
                    beta1=rng.uniform(1.0, 2.0), augmented=True, n_top=max(1, R // 32))
        if family == "max3cut":
            case.update(rule=rule)
        else:
            K = rng.choice([2, 3, 3, 4])
            case.update(K=K, potts_rule=rng.choice([pamc.POTTS_SOFTMAX, pamc.POTTS_CASCADE]) if K == 3 else
                        pamc.POTTS_SOFTMAX, gamma=1.0)
        return case
    if family == "dense_random":
        n = _odd(rng, _log_int(rng, 1000, 60000))
        return dict(family=family, n=n, R=min(R, 512), steps=max(2, min(30, int(1.2e11 / n / n))), sweeps=1, scale0=0.1,
                    scale1=3.0, rule=rule)
    if family == "dense_i8":
        n = _odd(rng, _log_int(rng, 200, 6000))
        return dict(family=family, n=n, jmax=rng.choice([1, 7, 100]), R=min(R, 512), steps=12, sweeps=rng.randint(1, 3),
                    scale0=0.1, scale1=3.0, rule=rule)
    if family == "batch":
        return dict(family=family, count=rng.randint(4, 64), n_min=200, n_max=2000, R=64 * rng.randint(1, 6), steps=30,
                    sweeps=rng.randint(1, 5), beta0=0.1, beta1=3.0)
    if family == "served":
        return dict(family=family, count=rng.randint(4, 32), n_min=800, n_max=20000, R=64 * rng.randint(1, 8), steps=20,
                    sweeps=rng.randint(1, 5), beta0=0.1, beta1=3.0)
    return dict(family=family, width=rng.randint(20, 140), height=rng.randint(20, 140), R=min(R, 1024),
                nbins=rng.randint(16, 128))


# ------------------------------------------------------------------ inputs
def _csr(n, u, v, w):
    src, dst, ww = np.concatenate([u, v]), np.concatenate([v, u]), np.concatenate([w, w])
    order = np.lexsort((dst, src))
    ptr = np.zeros(n + 1, np.int64)
    np.cumsum(np.bincount(src, minlength=n), out=ptr[1:])
    return SimpleNamespace(n=n, row_ptr=ptr.astype(np.int32), col=dst[order].astype(np.int32),
                           w=ww[order].astype(np.int32))


def _gnm(n, m, weights, seed):
    """m distinct edges, uniform over all pairs; weights 1, +-1, or +-1..1000."""
    rng = np.random.default_rng(seed)
    total = n * (n - 1) // 2
    if 3 * m > total:
        code = rng.choice(total, size=m, replace=False)
    else:
        code = np.unique(rng.integers(0, total, size=m + m // 2))
        while code.size < m:
            code = np.unique(np.concatenate([code, rng.integers(0, total, size=m)]))
        code = rng.permutation(code)[:m]
    # pair k = v (v - 1) / 2 + u with u < v
    v = ((1 + np.sqrt(1.0 + 8.0 * code)) / 2).astype(np.int64)
    v -= v * (v - 1) // 2 > code
    v += (v + 1) * v // 2 <= code
    u = code - v * (v - 1) // 2
    if weights == "one":
        w = np.ones(m, np.int32)
    elif weights == "pm1":
        w = 2 * rng.integers(0, 2, size=m) - 1
    else:
        w = rng.integers(1, 1001, size=m) * (2 * rng.integers(0, 2, size=m) - 1)
    return _csr(n, u, v, w)


def _torus(width, height, seed):
    """Periodic grid with +-1 weights, vertex id y * width + x."""
    rng = np.random.default_rng(seed)
    y, x = np.divmod(np.arange(width * height), width)
    u = np.concatenate([y * width + x] * 2)
    v = np.concatenate([y * width + (x + 1) % width, (y + 1) % height * width + x])
    return _csr(width * height, u, v, 2 * rng.integers(0, 2, size=u.size) - 1)


def _requests(case, seed):
    """Graphs of a request stream: n log-uniform, in turn a random graph of
    average degree 4 to 50 and a torus of even sides.  The sizes belong to
    the case, the graphs to the seed."""
    sizes, rng = np.random.default_rng(case["count"]), np.random.default_rng(seed)
    graphs = []
    for i in range(case["count"]):
        n = int(round(math.exp(sizes.uniform(math.log(case["n_min"]), math.log(case["n_max"])))))
        if i % 2 == 0:
            m = min(int(round(n * sizes.uniform(4.0, 50.0) / 2)), n * (n - 1) // 2)
            graphs.append(_gnm(n, m, "one", int(rng.integers(2**31))))
        else:
            h = max(4, 2 * int(round(math.sqrt(n / 2) / 2)))
            graphs.append(_torus(max(4, 2 * int(round(n / (2 * h)))), h, int(rng.integers(2**31))))
    return graphs


def _population(case, seed):
    """A population as resampling leaves it: families of a common ancestor,
    each member a few per cent of its spins away from it."""
    rng = np.random.default_rng(seed)
    n, R = case["width"] * case["height"], case["R"]
    ancestors = 2 * rng.integers(0, 2, size=(max(2, R // 16), n), dtype=np.int8) - 1
    member = ancestors[np.sort(rng.integers(0, ancestors.shape[0], size=R))]
    away = rng.random((R, 1), dtype=np.float32) * 0.1
    return np.where(rng.random((R, n), dtype=np.float32) < away, -member, member).astype(np.int8)


def _int8_couplings(case, seed):
    rng = np.random.default_rng(seed)
    n, j = case["n"], case["jmax"]
    up = np.triu(rng.integers(-j, j + 1, size=(n, n), dtype=np.int8), 1)
    return up + up.T


def _betas(case):
    if "beta0" in case:
        scale = 100.0 ** -1 if case.get("weights") == "wide" else 1.0
        return case["beta0"] * scale, case["beta1"] * scale
    size = math.sqrt(case["n"]) * math.sqrt(case.get("jmax", 1) * (case.get("jmax", 1) + 1) / 3 if "jmax" in case else 1)
    return case["scale0"] / size, case["scale1"] / size


def _schedule(case):
    b0, b1 = _betas(case)
    steps = case["steps"]
    kw = dict(beta0=b0, dbeta=(b1 - b0) / (steps - 1), steps=steps, sweeps=case["sweeps"])
    if case.get("augmented"):
        kw.update(augmented=1, z_rst=400, n_top=case["n_top"], mis_trials=4, tau=25)
    return pamc.schedule(**kw)


# --------------------------------------------------------------- the cases
def prepare(case, seed):
    """The instance (or server) a program holds, built from inputs of this
    seed, and its schedule."""
    family, R = case["family"], case.get("R")
    st = SimpleNamespace(case=case, seed=1000003 * seed + 17)
    rule = RULES[case.get("rule", "heatbath")]
    if family in ("gnm", "loop"):
        st.inst = pamc.Instance.csr(_gnm(case["n"], case["m"], case["weights"], seed), replicas=R, seed=st.seed, rule=rule)
    elif family == "torus":
        st.inst = pamc.Instance.csr(_torus(case["width"], case["height"], seed), replicas=R, seed=st.seed, rule=rule)
    elif family == "max3cut":
        st.inst = pamc.Instance.max3cut(_gnm(case["n"], case["m"], "one", seed), replicas=R, seed=st.seed, rule=rule)
    elif family == "potts":
        st.inst = pamc.Instance.potts(_gnm(case["n"], case["m"], "one", seed), case["K"], replicas=R, seed=st.seed,
                                      potts_rule=case["potts_rule"], gamma=case["gamma"])
    elif family == "dense_random":
        st.inst = pamc.Instance.dense_random(case["n"], seed, replicas=R, seed=st.seed, rule=rule)
    elif family == "dense_i8":
        st.inst = pamc.Instance.dense(_int8_couplings(case, seed), replicas=R, seed=st.seed, rule=rule)
    elif family == "batch":
        st.insts = [pamc.Instance.csr(g, replicas=R, seed=st.seed + i) for i, g in enumerate(_requests(case, seed))]
    elif family == "served":
        st.graphs = _requests(case, seed)
        st.server = pamc.Server(16 << 30, 256, replicas=R)
    else:
        st.inst = pamc.Instance.csr(_torus(case["width"], case["height"], seed), replicas=R, seed=st.seed)
        st.inst.set_state(_population(case, seed))
    if family != "diversity":
        st.sched = _schedule(case)
    return st


def _result(r):
    return [r.best_cut, r.best_energy, r.steps_run, r.n_cluster_moves, r.n_reheats, r.n_reversals, r.n_restarts]


def _energies(inst):
    """Energy and ancestor of every replica (the C call takes NULL for the
    spins and fields, which a program of this size leaves on the device)."""
    energies, lineage = np.zeros(inst.R, np.int64), np.zeros(inst.R, np.int32)
    status = pamc.lib.pamc_get_state(inst.h, None, None, energies.ctypes.data, lineage.ctypes.data)
    if status != pamc.PAMC_OK:
        raise pamc.PamcError(status, pamc.lib.pamc_last_error().decode())
    return energies, lineage


def run(st):
    case = st.case
    family = case["family"]
    if family == "diversity":
        counts, mean = st.inst.pair_distance_hist(case["nbins"])
        return dict(counts=counts, mean=mean)
    if family == "batch":
        for i, inst in enumerate(st.insts):
            inst.reset(st.seed + i)
        results = pamc.anneal_batch(st.insts, [st.sched] * len(st.insts))
        ends = [_energies(i) for i in st.insts]
        return dict(results=np.array([_result(r) for r in results]), spins=np.concatenate([i.best()[2] for i in st.insts]),
                    lnq=np.stack([i.trace(case["steps"])["lnq"] for i in st.insts]),
                    energies=np.stack([e for e, _ in ends]), lineage=np.stack([f for _, f in ends]))
    if family == "served":
        tickets = [st.server.submit(g, st.seed + i, st.sched) for i, g in enumerate(st.graphs)]
        st.server.drain()
        done = [st.server.poll(t, spins=True) for t in tickets]
        for t in tickets:
            st.server.forget(t)
        return dict(results=np.array([_result(r) for r, _ in done]), spins=np.concatenate([s for _, s in done]),
                    lnq=np.array([r.sum_lnq for r, _ in done]))
    inst = st.inst
    inst.reset(st.seed)
    if family == "loop":
        b0, b1 = _betas(case)
        delta = (b1 - b0) / (case["steps"] - 1)
        lnq = []
        for k in range(case["steps"]):
            if k:
                lnq.append(inst.resample(delta))
            inst.sweep(b0 + k * delta, case["sweeps"])
            inst.update_best()
        cut, energy, spins = inst.best()
        energies, lineage = _energies(inst)
        return dict(result=np.array([cut, energy]), spins=spins, lnq=np.array(lnq), energies=energies, lineage=lineage)
    res = inst.anneal(st.sched)
    _, _, spins = inst.best()
    trace = inst.trace(case["steps"])
    out = dict(result=np.array(_result(res)), spins=spins, mstar=trace["mstar"], beta=trace["beta"], lnq=trace["lnq"],
               events=trace["events"])
    if family == "max3cut":
        out["cut3"], out["labels"] = inst.max3cut_decode()
    if case.get("snapshot"):
        out["population"], out["fields"], out["energies"], out["lineage"] = inst.state()
    else:
        out["energies"], out["lineage"] = _energies(inst)
    return out


def exact(case, seed):
    """Outputs with a value in closed form: the pair-distance histogram and
    the inverse temperatures of a plain schedule."""
    family = case["family"]
    if family == "diversity":
        s = _population(case, seed).astype(np.float64)
        R, n = s.shape
        i, j = np.triu_indices(R, 1)
        d = (n - (s @ s.T)[i, j].astype(np.int64)) // 2
        d = np.minimum(d, n - d)
        bins = np.minimum(case["nbins"] - 1, 2 * case["nbins"] * d // n)
        return dict(counts=np.bincount(bins, minlength=case["nbins"]), mean=d.sum() / (n * len(d)))
    if family in ("loop", "batch", "served") or case.get("augmented"):
        return None
    b0, b1 = _betas(case)
    delta = (b1 - b0) / (case["steps"] - 1)
    out = dict(result=None, spins=None, mstar=None, lnq=None, events=None, energies=None, lineage=None,
               beta=np.cumsum(np.concatenate([[b0], np.full(case["steps"] - 1, delta)])))
    if family == "max3cut":
        out.update(cut3=None, labels=None)
    if case.get("snapshot"):
        out.update(population=None, fields=None)
    return out


# ------------------------------------------------------------------- work
# One visit of a spin cannot do without its share of a Philox4x32-10 block
# (ten rounds of two products and four xors for four visits: 15 operations),
# the compare and update (5), and a multiply-add per neighbour.  A beta step
# reads and writes the population once (a byte per spin: resampling); the
# couplings are read once per sweep where they do not fit the caches (dense),
# else once.
def _sparse_work(n, nnz, R, steps, sweeps, words=1):
    return dict(bytes=steps * 2.0 * n * R + 8.0 * nnz, flops=steps * sweeps * R * ((5.0 + 15.0 * words) * n + 2.0 * nnz))


def work(case):
    family = case["family"]
    if family == "diversity":
        n, R = case["width"] * case["height"], case["R"]
        return dict(bytes=float(n * R), flops=1.0 * R * (R - 1) * n)
    R, steps, sweeps = case["R"], case["steps"], case["sweeps"]
    if family in ("gnm", "loop"):
        return _sparse_work(case["n"], 2 * case["m"], R, steps, sweeps)
    if family == "torus":
        n = case["width"] * case["height"]
        return _sparse_work(n, 4 * n, R, steps, sweeps)
    if family == "max3cut":
        n, m = case["n"], case["m"]
        return _sparse_work(3 * n + 1, 2 * (6 * n + 3 * m), R, steps, sweeps)
    if family == "potts":
        cascade = case["potts_rule"] == pamc.POTTS_CASCADE
        return _sparse_work(case["n"], 2 * case["m"], R, steps, sweeps, words=2 if cascade else case["K"])
    if family in ("dense_random", "dense_i8"):
        n = case["n"]
        return dict(bytes=steps * sweeps * 1.0 * n * n + steps * 2.0 * n * R,
                    flops=steps * sweeps * R * (2.0 * n * n + 20.0 * n))
    # batch and served: the mean size of a log-uniform n, half the graphs of
    # mean degree 27, half of degree 4
    lo, hi = case["n_min"], case["n_max"]
    n = (hi - lo) / math.log(hi / lo) * case["count"]
    return _sparse_work(n, 15.5 * n, R, steps, sweeps)
