"""The server's memory budget against what the device reports: many small
requests running at once hold no more than the budget."""
import pytest

import synth

pytestmark = pytest.mark.gpu


def test_small_requests_stay_within_the_budget():
    import torch
    from paper_2606_25203_amd import pamc
    budget, count = 24 << 20, 120
    sched = pamc.schedule(beta0=0.1, dbeta=0.1, steps=8, sweeps=2, augmented=1, n_top=2, mis_trials=2)
    graphs = [synth.random_graph(60 + i % 7, 150, i) for i in range(count)]

    def running(n):
        srv = pamc.Server(budget, 256, replicas=64)
        tickets = [srv.submit(g, 7 + i, sched) for i, g in enumerate(graphs[:n])]
        active, _ = srv.tick(1)
        while active < n:  # requests still being prepared
            active, _ = srv.tick(1)
            assert active, "all done before all were admitted"
        free = torch.cuda.mem_get_info()[0]
        counted = srv.stats()["in_use_bytes"]
        srv.drain()
        for i, t in enumerate(tickets):
            assert srv.poll(t).steps_run == 8, i
        srv.close()
        return free, counted

    print("case many small requests", flush=True)
    running(2)  # the device's own allocations at first use
    base, few = running(1)
    free, counted = running(count)
    held = base - free
    print(f"  counted {counted} bytes, held {held}", flush=True)
    assert counted <= budget and held <= budget - few
