"""The batched anneal with fixed scratch near the scratch's end: instances that
could sweep bit-packed are refused no earlier than the same ones kept from it
(their launches' maps and phase records are given up when they do not fit),
and give the results of the allocating call on either side."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pamc():
    from paper_2606_25203_amd import pamc as p
    return p


def make(pamc):
    small = synth.torus(6, 4, 1)
    big = synth.torus(100, 200, 2)
    return [pamc.Instance.csr(big, replicas=64, seed=1)] + \
        [pamc.Instance.csr(small, replicas=64, seed=2 + i) for i in range(40)]


def schedules(pamc, sweeps, steps):
    # the big instance's cluster scratch leaves some 200 KB for the rest, of
    # which its class orders take 8 bytes a sweep (and phase records 32 more)
    aug = dict(beta0=0.1, dbeta=0.05, augmented=1, z_rst=60, n_top=63, mis_trials=13, win_short=5, win_long=8, tau=4)
    plain = dict(beta0=0.1, dbeta=0.05, steps=steps, sweeps=1)
    return [pamc.schedule(steps=steps, sweeps=sweeps, **aug)] + [pamc.schedule(**plain)] * 40


def accepted(pamc, insts, sweeps):
    try:
        pamc.anneal_batch_noalloc(insts, schedules(pamc, sweeps, 0))
        return True
    except pamc.PamcError as e:
        assert e.status == pamc.PAMC_ERR_UNSUPPORTED and "scratch" in str(e)
        return False


def test_refused_no_earlier(pamc, monkeypatch):
    monkeypatch.setenv("PAMC_BITS", "0")
    other = make(pamc)
    monkeypatch.setenv("PAMC_BITS", "1")
    insts = make(pamc)
    monkeypatch.delenv("PAMC_BITS")
    print("case noalloc limits", flush=True)
    assert accepted(pamc, other, 1) and not accepted(pamc, other, 200_000)
    lo, hi = 1, 200_000  # the most sweeps that fit without bit-packed launches
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (mid, hi) if accepted(pamc, other, mid) else (lo, mid)
    assert lo > 1000
    for sweeps in list(range(64, lo, 48)) + [lo - 1, lo]:
        assert accepted(pamc, insts, sweeps), sweeps
    assert not accepted(pamc, insts, lo + 64)
    for i in other + insts:
        i.close()


@pytest.mark.parametrize("sweeps", [40, 3000])
def test_same_results_either_way(pamc, monkeypatch, sweeps):
    """40 sweeps: phase records in the instance's own buffer; 3,000: in the
    scratch, or given up."""
    monkeypatch.setenv("PAMC_BITS", "1")
    print(f"case noalloc results, {sweeps} sweeps", flush=True)
    a, b = make(pamc)[:8], make(pamc)[:8]
    ra = pamc.anneal_batch(a, schedules(pamc, sweeps, 2)[:8])
    rb = pamc.anneal_batch_noalloc(b, schedules(pamc, sweeps, 2)[:8])
    for x, y, p, q in zip(ra, rb, a, b):
        assert (x.best_cut, x.sum_lnq, x.steps_run) == (y.best_cut, y.sum_lnq, y.steps_run)
        assert all(np.array_equal(m, n) for m, n in zip(p.state(), q.state()))
        p.close()
        q.close()


def test_diversity_samples_of_many_replicas(pamc, monkeypatch):
    """The largest population's diversity samples: a launch map of at most a
    word per replica (the scratch is filled by class orders of 8 bytes a sweep,
    cut in pieces of 256), and the mean of all pairs."""
    monkeypatch.setenv("PAMC_BITS", "0")
    R = 16384
    print("case diversity samples, R = 16384", flush=True)
    inst = pamc.Instance.csr(synth.torus(6, 4, 1), replicas=R, seed=1)

    def most_sweeps(dh_every):
        lo, hi = 1, 1 << 22
        while hi - lo > 1:
            mid = (lo + hi) // 2
            try:
                pamc.anneal_batch_noalloc([inst], [pamc.schedule(steps=0, sweeps=mid, dh_every=dh_every)])
                lo = mid
            except pamc.PamcError as e:
                assert e.status == pamc.PAMC_ERR_UNSUPPORTED
                hi = mid
        return lo

    assert 8 * (most_sweeps(0) - most_sweeps(1)) <= 8 * R + 512
    inst.anneal(pamc.schedule(beta0=0.1, dbeta=0.2, steps=3, sweeps=2, dh_every=1))
    dh = pamc.pamc_get_dh_trace(inst.h, 3)
    assert dh[2] == inst.pair_distance() and 0 < dh[0] <= 0.5
    s = inst.state()[0].astype(np.int64)
    d = (s.shape[1] - s[:512] @ s.T) // 2  # of the first 512 replicas to all
    d = np.minimum(d, s.shape[1] - d).sum() / s.shape[1] / (512 * (R - 1))
    assert abs(d - dh[2]) < 0.05
    inst.close()
