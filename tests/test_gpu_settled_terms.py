"""GPU: settled sweeps of problems whose products mix short and long records (x^2 y z w: three other factors
for x, four for y) against the oracle, in plain runs, batches and served chunks, with schedules that cool,
warm up again and cool."""
import numpy as np
import pytest

import oracle
from paper_2511_17245_amd import inputs as I
from paper_2511_17245_amd import sa
from tests import parity
from tests.test_gpu_settled import run

pytestmark = pytest.mark.gpu

RULES = [sa.METROPOLIS, sa.HEAT_BATH, sa.OPT_METROPOLIS, sa.HEAT_BATH_CLOSED]


def problem(kind, n=40, seed=3):
    g = np.random.Generator(np.random.PCG64([seed, n]))
    def coef():
        return int(g.integers(1, 6)) * (1 if g.integers(2) else -1)
    def some(m):
        return [int(x) for x in g.choice(n, m, replace=False)]
    terms = [(coef(), [i]) for i in range(n)]
    for _ in range(2 * n):
        a, b, c, d = some(4)
        if kind == "one_square":       # x^2 y z w
            terms.append((coef(), [a, a, b, c, d]))
        elif kind == "two_squares":    # x^2 y^2 z
            terms.append((coef(), [a, a, b, b, c]))
        else:                          # those among terms of degree two to four, some of them squares
            terms.append((coef(), [[a, a, b, c, d], [a, a, b, b, c], [a, b], [a, a, b], [a, b, b, c]][g.integers(5)]))
    return I.from_terms(n, terms, -2, 3)


def schedule(prob, sweeps=60):
    """Cooled until nothing moves, warmed past the start, cooled again."""
    b = oracle.Poly(prob).schedule(sweeps)[0]
    return np.concatenate([b, b[10::-5], b[::2]])


@pytest.mark.parametrize("kind", ["one_square", "two_squares", "mixed"])
@pytest.mark.parametrize("rule", RULES)
def test_every_sweep_against_the_oracle(kind, rule):
    prob = problem(kind)
    P = oracle.Poly(prob)
    beta = schedule(prob)
    reads, seed = 6, 0x5EA + rule
    zo, eo, ho = P.anneal(rule, beta, reads, seed, trace=True)
    for G in (1, 2, 0):
        z, e, h = run(prob, rule, beta, reads, seed, G)

        def explain(i):
            def after(s, zb):
                return run(prob, rule, beta, i + 1, seed, G, np.tile(zb, (i + 1, 1)), s, s + 1, trace=False)[0][i]
            return parity.localise(P, rule, beta, seed, 0, i, h[i], after)

        parity.check(f"terms {kind} rule {rule} G {G}", reads,
                     lambda i: np.array_equal(z[i], zo[i]) and e[i] == eo[i] and np.array_equal(h[i], ho[i]), explain)


@pytest.mark.parametrize("rule", RULES)
def test_squares_on_fixed_variables_only(rule):
    """Cached coefficients without one of a square, and fixed variables that have a square."""
    g = np.random.Generator(np.random.PCG64(8))
    terms = [(int(g.integers(1, 9)) * (1 if i % 2 else -1), [i, i + 1]) for i in range(39)]
    terms += [(int(g.integers(-9, 10)) or 1, [i]) for i in range(40)] + [(2, [0, 0, 1]), (3, [7, 7]), (-2, [21, 21, 20])]
    prob = I.from_terms(40, terms, -2, 3)
    for k, v in ((0, 2), (7, -1), (21, 3)):
        prob.lower[k] = prob.upper[k] = v
    P = oracle.Poly(prob)
    beta = schedule(prob)
    for G in (1, 2):
        z, e, h = run(prob, rule, beta, 4, 0xF1 + rule, G)
        zo, eo, ho = P.anneal(rule, beta, 4, 0xF1 + rule, trace=True)
        assert np.array_equal(z, zo) and np.array_equal(e, eo) and np.array_equal(h, ho)


def items():
    out = []
    for i, (kind, rule) in enumerate((k, r) for k in ("one_square", "two_squares", "mixed") for r in RULES):
        prob = problem(kind, 30 + 3 * i, 50 + i)
        beta = schedule(prob, 50)
        out.append(I.Workload(prob, rule, len(beta), 5, 70 + i, i, beta=beta))
    return out


def check(label, got, work):
    for i, (w, (z, e)) in enumerate(zip(work, got)):
        P = oracle.Poly(w.problem)
        assert all(int(e[j]) == P.energy(z[j]) for j in range(w.n_reads)), f"{label} {i}: energies of the states"
        zp, ep, _ = run_alone(w)
        assert np.array_equal(z, zp) and np.array_equal(e, ep), f"{label} {i}"


def run_alone(w):
    import torch
    plan = sa.Plan(w.problem, w.rule)
    z = torch.empty((w.n_reads, w.problem.n_vars), dtype=torch.int32, device="cuda")
    e = torch.empty(w.n_reads, dtype=torch.int64, device="cuda")
    h = torch.empty((w.n_reads, w.n_sweeps), dtype=torch.int64, device="cuda")
    plan.run_device(w.n_sweeps, w.n_reads, w.seed, z, e, beta=w.beta, stream=torch.cuda.current_stream().cuda_stream,
                    instance_id=w.instance_id, waves_per_replica=1, trace=h)
    torch.cuda.synchronize()
    plan.close()
    return z.cpu().numpy(), e.cpu().numpy(), h


@pytest.mark.parametrize("graph", [False, True])
def test_batch(graph):
    work = items()
    b = sa.Batch(work, use_graph=graph)
    for _ in range(2):
        b.run()
        check("batch", b.results(), work)
    b.close()


@pytest.mark.parametrize("chunk", [7, 30])
def test_served_chunks(chunk):
    work = items()
    srv = sa.Server(chunk_sweeps=chunk)
    tickets = [srv.submit(w) for w in work]
    assert all(srv.wait(t)["status"] == sa.OK for t in tickets)
    check("served", [srv.result(t) for t in tickets], work)
    srv.close()
