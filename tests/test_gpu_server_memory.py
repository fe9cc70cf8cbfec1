"""GPU: the server's memory in use holds what requests and their plans keep on the device, the lists built for
the faster kernels among them; a budget that holds a request without them still serves it."""
import time

import numpy as np
import pytest

from paper_2511_17245_amd import inputs as I
from paper_2511_17245_amd import sa

pytestmark = pytest.mark.gpu


def in_use(work, **kw):
    """Memory in use while the request runs; 0 once it is done."""
    srv = sa.Server(chunk_sweeps=1, **kw)
    t = srv.submit(work)
    most, deadline = 0, time.time() + 60
    while not srv.poll(t)[0] and time.time() < deadline:
        st = srv.stats()
        most = max(most, st["mem_in_use"])
    assert srv.wait(t)["status"] == sa.OK
    z, e = srv.result(t)
    after = srv.stats()["mem_in_use"]
    srv.close()
    return most, after, z, e


def test_memory_in_use():
    prob = I.erdos_renyi_quio(3000, 8.0, -20, 19, 10, 10, np.random.Generator(np.random.PCG64(31)))
    edges = int((np.diff(prob.term_ptr) == 2).sum())
    reads = 64
    heat, after, z, e = in_use(I.Workload(prob, sa.HEAT_BATH, 20000, reads, 5, 1))
    metro, _, _, _ = in_use(I.Workload(prob, sa.METROPOLIS, 3000, reads, 5, 1))
    assert after == 0
    # states, energies and next sweeps; couplings and one list of the variables, as records of 32 bytes
    assert min(heat, metro) >= reads * (4 * prob.n_vars + 8 + 4) + 2 * edges * 8 + prob.n_vars * 32
    # the lane kernel's records on top, four bytes each
    assert heat - metro >= 2 * edges * 4
    # a budget for what the request cannot do without (schedule, states, energies, instance), in whole 256 bytes
    plan = sa.Plan(prob, sa.HEAT_BATH)
    budget = sum((b + 255) // 256 * 256 for b in (8 * 20000, reads * 4 * prob.n_vars, reads * 8)) + plan.info()["device_bytes"]
    plan.close()
    assert budget < heat
    _, _, z2, e2 = in_use(I.Workload(prob, sa.HEAT_BATH, 20000, reads, 5, 1), mem_budget_bytes=budget)
    assert np.array_equal(z, z2) and np.array_equal(e, e2)
