"""Requests submitted to one server by several threads at once, of materials that do and do not
share a kernel: every ticket is distinct, every request completes, and each result is bitwise the
request decoded alone, whatever the order in which launches group them."""
import threading

import numpy as np
import pytest

from paper_2305_02678_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["f16", "f32"])
def test_concurrent_submissions(precision):
    import torch
    from paper_2305_02678_amd import nam
    ctx = nam.Context(0)
    server = nam.Server(ctx, n_streams=3, max_tile=2048)
    mats = []
    for k, (C, hidden) in enumerate([(16, [64] * 3), (8, [64] * 3), (16, [32] * 2)]):
        r = wl.rngs(90 + k)
        m = nam.Material.from_workload(ctx, wl.make_material(r[0], r[1], 64, 64, C, 4, hidden))
        if precision == "f16":
            m.set_precision(nam.F16)
        mats.append((m, server.add_material(m)))
    rng = np.random.default_rng(5)
    jobs = [[] for _ in range(4)]
    for k in range(80):
        q = nam.to_device(wl.uniform_queries(rng, int(rng.integers(0, 5000)), -0.5, 3.5))
        jobs[k % 4].append((int(rng.integers(0, 3)), q, torch.full((len(q[1]), 3), -1.0, device="cuda")))
    torch.cuda.synchronize()
    tickets = [[] for _ in range(4)]

    def run(t):
        for m, q, rgb in jobs[t]:
            tickets[t].append(server.submit(mats[m][1], *q, rgb))

    threads = [threading.Thread(target=run, args=(t,)) for t in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    server.wait_all()
    every = [x for t in tickets for x in t]
    assert len(set(every)) == 80 and all(server.poll(x)[0] for x in every)
    assert server.stats()["completed"] == 80
    for m, q, rgb in (j for t in jobs for j in t):
        assert torch.equal(rgb, nam.decode(mats[m][0], *q))
    server.close()


def test_reset_keeps_the_buffers_of_waiting_requests():
    """A request that has not finished when the statistics are reset keeps its tensors, whatever the
    caller does with its own references; a finished one gives them back."""
    import torch
    from paper_2305_02678_amd import nam
    ctx = nam.Context(0)
    server = nam.Server(ctx, n_streams=2, max_tile=2048)
    r = wl.rngs(94)
    m = nam.Material.from_workload(ctx, wl.make_material(r[0], r[1], 64, 64, 16, 4, [32] * 2))
    mid = server.add_material(m)
    q = nam.to_device(wl.uniform_queries(r[2], 3000, -0.5, 3.5))
    first, late = (torch.full((3000, 3), -1.0, device="cuda") for _ in range(2))
    a = server.submit(mid, *q, first)
    server.wait_all()
    b = server.submit(mid, *q, late, arrival_s=0.3)
    server.reset_stats()
    assert a not in server._keep and b in server._keep
    with pytest.raises(nam.NamError):
        server.poll(a)
    server.wait_all()
    assert server.poll(b)[0] and torch.equal(late, nam.decode(m, *q))
    server.reset_stats()
    assert not server._keep
    server.close()
