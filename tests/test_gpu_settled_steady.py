"""GPU: runs at one temperature, where replicas settle by chance or not at all: the hand-over to the settled
kernel, all replicas together, against the oracle sweep by sweep; more replicas than run at once; the same plan
on two streams."""
import numpy as np
import pytest

import oracle
from paper_2511_17245_amd import inputs as I
from paper_2511_17245_amd import sa
from tests import parity
from tests.test_gpu_settled import problem, run

pytestmark = pytest.mark.gpu

RULES = [sa.METROPOLIS, sa.HEAT_BATH, sa.OPT_METROPOLIS, sa.HEAT_BATH_CLOSED]


@pytest.mark.parametrize("kind", ["dense", "pairs", "huio", "long"])
@pytest.mark.parametrize("rule", RULES)
def test_one_temperature(kind, rule):
    prob = problem(kind)
    P = oracle.Poly(prob)
    b = P.schedule(101)[0]
    for frac, n_sweeps in ((30, 60), (45, 70), (60, 90)):
        beta = np.full(n_sweeps, b[frac])
        reads, seed = 16, 0x57EAD + rule + frac
        zo, eo, ho = P.anneal(rule, beta, reads, seed, trace=True)
        for G in (0, 1, 2):
            if kind == "dense" and G == 2:
                continue
            z, e, h = run(prob, rule, beta, reads, seed, G)

            def explain(i):
                def after(s, zb):
                    return run(prob, rule, beta, i + 1, seed, G, np.tile(zb, (i + 1, 1)), s, s + 1, trace=False)[0][i]
                return parity.localise(P, rule, beta, seed, 0, i, h[i], after)

            parity.check(f"steady {kind} rule {rule} at {frac} G {G}", reads,
                         lambda i: np.array_equal(z[i], zo[i]) and e[i] == eo[i] and np.array_equal(h[i], ho[i]), explain)


@pytest.mark.parametrize("rule", [sa.METROPOLIS, sa.OPT_METROPOLIS])
def test_more_replicas_than_run_at_once(rule):
    prob = I.dense_quio(40, -3, 4, 10, 10, np.random.Generator(np.random.PCG64(12)))
    P = oracle.Poly(prob)
    beta = P.schedule(80)[0]
    zo, eo = P.anneal(rule, beta, 12000, 5)
    z, e, _ = run(prob, rule, beta, 12000, 5, 0, trace=False)
    assert np.array_equal(z, zo) and np.array_equal(e, eo)


def test_one_plan_on_two_streams():
    import torch
    prob = I.random_huio(600, 4800, [2, 3, 4], -8, 8, 5, np.random.Generator(np.random.PCG64(13)))
    beta = oracle.Poly(prob).schedule(200)[0]
    plan = sa.Plan(prob, sa.METROPOLIS)
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    bufs = [(torch.empty((64, 600), dtype=torch.int32, device="cuda"), torch.empty(64, dtype=torch.int64, device="cuda"))
            for _ in range(4)]
    torch.cuda.synchronize()
    for i, (z, e) in enumerate(bufs[:2]):
        plan.run_device(200, 64, 40 + i, z, e, beta=beta, stream=streams[0].cuda_stream)
        torch.cuda.synchronize()
    for i, (z, e) in enumerate(bufs[2:]):
        plan.run_device(200, 64, 40 + i, z, e, beta=beta, stream=streams[i].cuda_stream)
    torch.cuda.synchronize()
    for a, b in zip(bufs[:2], bufs[2:]):
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    plan.close()


def test_replicas_that_settle_near_the_end():
    """Some settle while they may still leave, others after: none leaves, or the settled kernel's sweeps come on top
    of the run (a seventh of it).  Against the same run in pieces of 40 sweeps, which leave too little to hand over;
    two runs of one kind differ by less than 0.01."""
    import time

    import torch
    n, S, reads = 3000, 200, 512
    prob = I.erdos_renyi_quio(n, 8, 0, 3, 10, 10, np.random.Generator(np.random.PCG64(3)))
    plan = sa.Plan(prob, sa.OPT_METROPOLIS)
    bufs = [(torch.empty((reads, n), dtype=torch.int32, device="cuda"), torch.empty(reads, dtype=torch.int64, device="cuda"))
            for _ in range(3)]

    def timed(pieces):
        best = 1e9
        for _ in range(4):
            torch.cuda.synchronize()
            t = time.perf_counter()
            zi = None
            for i, (s0, s1) in enumerate(pieces):
                z, e = bufs[i % 3]
                plan.run_device(S, reads, 5, z, e, sweep_begin=s0, sweep_end=s1, init_states=zi,
                                stream=torch.cuda.current_stream().cuda_stream)
                zi = z
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t)
        return best, z.clone(), e.clone()

    whole, z, e = timed([(0, S)])
    parts, zp, ep = timed([(s, s + 40) for s in range(0, S, 40)])
    plan.close()
    print(f"whole {1e3 * whole:.2f} ms, in pieces {1e3 * parts:.2f} ms")
    assert torch.equal(z, zp) and torch.equal(e, ep)
    assert whole < 1.06 * parts
