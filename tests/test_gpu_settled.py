"""GPU: runs whose replicas settle (the settled kernel takes the later sweeps, and the last launch
the replicas that warm up again) against the oracle, sweep by sweep, at tests/parity.py's bar."""
import numpy as np
import pytest

import oracle
from paper_2511_17245_amd import inputs as I
from paper_2511_17245_amd import sa
from tests import parity

pytestmark = pytest.mark.gpu

RULES = [sa.METROPOLIS, sa.HEAT_BATH, sa.OPT_METROPOLIS, sa.HEAT_BATH_CLOSED]


def rng(seed):
    return np.random.Generator(np.random.PCG64(seed))


def problem(kind):
    g = rng(77)
    if kind == "dense":            # coefficient cache, squares in one half of the variables
        return I.dense_quio(65, -4, 11, 10, 10, g)
    if kind == "dense_linear":     # no squares, int32 couplings, ranges past 512 values
        return I.fully_connected(40, 1, 400)
    if kind == "pairs":            # cached coefficients only; 64 k - 1 variables
        return I.erdos_renyi_quio(191, 6.0, -50, 50, 10, 20, g)
    if kind == "pairs_w2":
        return I.erdos_renyi_quio(129, 8.0, 0, 1, 10, 10, g)
    if kind == "huio":             # cached and margin variables together, powers up to four
        return I.random_huio(128, 900, [1, 2, 3, 4], -6, 13, 5, g)
    if kind == "huio_wide":        # W = 513: one past the weights kept in registers
        return I.random_huio(64, 260, [2, 3], -256, 256, 5, g)
    if kind == "long":             # terms with more than three other factors: margins, flat variables
        return I.multilinear(63, 7, 3)
    if kind == "big":              # coefficients past 32 bits: margins only
        p = I.random_huio(40, 200, [2, 3], -9, 9, 5, g)
        p.coef = p.coef * (1 << 33)
        return p
    raise ValueError(kind)


def run(prob, rule, beta, reads, seed, G, z_init=None, s0=0, s1=0, trace=True):
    import torch
    plan = sa.Plan(prob, rule)
    n_tr = (s1 or len(beta)) - s0
    z = torch.empty((reads, prob.n_vars), dtype=torch.int32, device="cuda")
    e = torch.empty(reads, dtype=torch.int64, device="cuda")
    h = torch.empty((reads, n_tr), dtype=torch.int64, device="cuda") if trace else None
    zi = None if z_init is None else torch.as_tensor(np.ascontiguousarray(z_init, np.int32), device="cuda")
    plan.run_device(len(beta), reads, seed, z, e, beta=beta, stream=torch.cuda.current_stream().cuda_stream,
                    sweep_begin=s0, sweep_end=s1, init_states=zi, waves_per_replica=G, trace=h)
    torch.cuda.synchronize()
    plan.close()
    return z.cpu().numpy(), e.cpu().numpy(), h.cpu().numpy().view(np.uint64) if trace else None


@pytest.mark.parametrize("kind", ["dense", "dense_linear", "pairs", "pairs_w2", "huio", "huio_wide", "long", "big"])
@pytest.mark.parametrize("rule", RULES)
def test_cooling_and_warming(kind, rule):
    """Cooled until nothing moves, warmed past the start, cooled again: every launch of the chain takes
    part.  Each sweep's state hash against the oracle's."""
    prob = problem(kind)
    P = oracle.Poly(prob)
    b = P.schedule(60)[0]
    beta = np.concatenate([b, b[10::-5], b[::2]])
    reads, seed = 6, 0x5E771ED + rule
    zo, eo, ho = P.anneal(rule, beta, reads, seed, trace=True)
    for G in (1, 2, 0):
        if kind.startswith("dense") and G == 2:
            continue
        z, e, h = run(prob, rule, beta, reads, seed, G)

        def explain(i):
            def after(s, zb):
                return run(prob, rule, beta, i + 1, seed, G, np.tile(zb, (i + 1, 1)), s, s + 1, trace=False)[0][i]
            return parity.localise(P, rule, beta, seed, 0, i, h[i], after)

        parity.check(f"settled {kind} rule {rule} G {G}", reads,
                     lambda i: np.array_equal(z[i], zo[i]) and e[i] == eo[i] and np.array_equal(h[i], ho[i]), explain)


@pytest.mark.parametrize("rule", RULES)
def test_resumed_and_without_allocations(rule):
    """A run resumed from its state after 50 of 80 sweeps, and sa_anneal_noalloc, end as the whole run."""
    import torch
    prob = problem("huio")
    beta = oracle.Poly(prob).schedule(80)[0]
    z, e, _ = run(prob, rule, beta, 5, 11, 2)
    zm, _, _ = run(prob, rule, beta, 5, 11, 2, s1=50)
    z2, e2, _ = run(prob, rule, beta, 5, 11, 2, z_init=zm, s0=50)
    assert np.array_equal(z, z2) and np.array_equal(e, e2)
    for G in (1, 2):
        zt = torch.empty((5, prob.n_vars), dtype=torch.int32, device="cuda")
        et = torch.empty(5, dtype=torch.int64, device="cuda")
        sa.anneal_device(prob, rule, 80, 5, 11, zt, et, beta=beta, waves_per_replica=G, no_alloc=True,
                         stream=torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert np.array_equal(z, zt.cpu().numpy()) and np.array_equal(e, et.cpu().numpy())


@pytest.mark.parametrize("sizes", [(100, 90), (100, 1500), (1500, 100, 4500, 120, 1600)])
@pytest.mark.parametrize("graph", [False, True])
def test_batch_groups_beside_each_other(sizes, graph):
    """One, two and three groups of settled replicas in one batch (by the LDS a replica takes): each
    problem ends as in a run of its own, in each of three runs of the batch."""
    items = [I.Workload(I.erdos_renyi_quio(n, 4.0, -3, 4, 10, 10, rng(n)), sa.METROPOLIS, 40, 3, 5 + i, i)
             for i, n in enumerate(sizes)]
    want = []
    for w in items:
        plan = sa.Plan(w.problem, w.rule)
        want.append(plan.run(w.n_sweeps, w.n_reads, w.seed, instance_id=w.instance_id)[:2])
        plan.close()
    b = sa.Batch(items, use_graph=graph)
    for _ in range(3):
        b.run()
        for (z, e), (zp, ep) in zip(b.results(), want):
            assert np.array_equal(z, zp) and np.array_equal(e, ep)
    b.close()
