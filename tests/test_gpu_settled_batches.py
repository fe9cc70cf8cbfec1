"""GPU: the hand-over between the ordinary and the settled kernel where it is hidden from plain runs' results: that
it takes place, and in batches and served chunks also back again (schedules that warm up), with teams of several waves
and several reads per task; dense teams of every rule in batches and resumed chunks."""
import numpy as np
import pytest

import oracle
from paper_2511_17245_amd import inputs as I
from paper_2511_17245_amd import sa
from tests import parity
from tests.test_gpu_parity import explainer
from tests.test_gpu_settled import problem

pytestmark = pytest.mark.gpu

RULES = [sa.METROPOLIS, sa.HEAT_BATH, sa.OPT_METROPOLIS, sa.HEAT_BATH_CLOSED]


def rng(seed):
    return np.random.Generator(np.random.PCG64(seed))


@pytest.mark.parametrize("kind", ["dense", "dense_linear", "pairs", "pairs_w2", "huio", "huio_wide", "long", "big"])
@pytest.mark.parametrize("rule", RULES)
def test_the_settled_kernel_takes_part(kind, rule):
    prob = problem(kind)
    plan = sa.Plan(prob, rule)
    for G in (1, 2):
        plan.run(93, 2, 1, waves_per_replica=G)
        assert plan.last_launch()["kernel_variant"] >= 10_000_000
        plan.run(8, 2, 1, waves_per_replica=G)      # too short to gain
        assert plan.last_launch()["kernel_variant"] < 10_000_000
    plan.close()


def test_pairs_in_two_goes_stay():
    """Pair problems of 10000 variables, one settled replica per CU: in 1.8 goes, not in two."""
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    prob = I.erdos_renyi_quio(10000, 4, 0, 3, 10, 10, rng(3))
    plan = sa.Plan(prob, sa.METROPOLIS)
    for reads, settled in ((cus * 9 // 5, True), (2 * cus, False)):
        plan.run(60, reads, 1)
        assert (plan.last_launch()["kernel_variant"] >= 10_000_000) == settled
    plan.close()


def warming(prob, sweeps):
    """Cooled, warmed past the start, cooled again."""
    b = oracle.Poly(prob).schedule(sweeps)[0]
    return np.concatenate([b, b[sweeps // 6::-3], b[::2]])


def items():
    out = []
    for i, rule in enumerate(RULES + [sa.METROPOLIS, sa.OPT_METROPOLIS]):
        n = 150 + 90 * i
        prob = I.random_huio(n, 4 * n, [2, 3], -5, 6, 5, rng(60 + i)) if i % 2 else I.random_huio(n, 3 * n, [1, 2], 0, 9, 5, rng(60 + i))
        beta = warming(prob, 60)
        out.append(I.Workload(prob, rule, len(beta), 7, 900 + i, i, beta=beta))
    return out


def check(label, got, work):
    for i, (w, (z, e)) in enumerate(zip(work, got)):
        P = oracle.Poly(w.problem)
        zo, eo = P.anneal(w.rule, w.beta, w.n_reads, w.seed, w.instance_id)
        assert all(int(e[j]) == P.energy(z[j]) for j in range(w.n_reads)), f"{label} {i}: energies of the states"
        parity.check(f"{label} {i}", w.n_reads, lambda j: e[j] == eo[j] and np.array_equal(z[j], zo[j]),
                     explainer(w.problem, P, w.rule, w.beta, w.seed, w.instance_id, G=1))


@pytest.mark.parametrize("graph", [False, True])
def test_batch_that_warms_up(graph):
    work = items()
    b = sa.Batch(work, use_graph=graph)
    assert 1 < b.info()["max_team"] <= 8
    for _ in range(2):
        b.run()
        check("warming batch", b.results(), work)
    b.close()


@pytest.mark.parametrize("chunk", [4, 17, 45])
def test_served_requests_that_warm_up(chunk):
    """The warm-up falls inside a chunk and across its end."""
    work = items()
    srv = sa.Server(chunk_sweeps=chunk)
    tickets = [srv.submit(w) for w in work]
    assert all(srv.wait(t)["status"] == sa.OK for t in tickets)
    check(f"served by {chunk}", [srv.result(t) for t in tickets], work)
    srv.close()


def test_dense_teams_in_batches_and_chunks():
    prob = I.dense_quio(1030, -3, 5, 10, 10, rng(44))
    prob.lower[::97] = prob.upper[::97]
    beta = oracle.Poly(prob).schedule(24)[0]
    beta = np.concatenate([beta[::2], beta[8::-3], beta[1::2]])
    work = [I.Workload(prob, rule, len(beta), 2, 70 + i, i, beta=beta) for i, rule in enumerate(RULES)]
    b = sa.Batch(work)
    assert b.info()["max_team"] > 1
    b.run()
    check("dense teams", b.results(), work)
    b.close()
    for chunk in (1, 5):
        srv = sa.Server(chunk_sweeps=chunk)
        tickets = [srv.submit(w) for w in work]
        assert all(srv.wait(t)["status"] == sa.OK for t in tickets)
        check(f"dense teams by {chunk}", [srv.result(t) for t in tickets], work)
        srv.close()
