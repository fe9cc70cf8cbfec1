"""GPU: dense problems annealed by a team of waves per replica, against the oracle sweep by sweep at
tests/parity.py's bar."""
import numpy as np
import pytest

import oracle
from paper_2511_17245_amd import inputs as I
from paper_2511_17245_amd import sa
from tests import parity

pytestmark = pytest.mark.gpu

RULES = [sa.METROPOLIS, sa.HEAT_BATH, sa.OPT_METROPOLIS, sa.HEAT_BATH_CLOSED]


def problem(kind):
    g = np.random.Generator(np.random.PCG64(123))
    if kind == "n1030":            # four columns per thread and a ragged end; some variables fixed
        p = I.dense_quio(1030, -3, 5, 10, 10, g)
        p.lower[::97] = p.upper[::97]
        return p
    if kind == "n1100_int32":      # couplings past int8; no squares in one half
        p = I.dense_quio(1100, 0, 9, 900, 500, g)
        keep = np.ones(p.n_terms, bool)
        deg = np.diff(p.term_ptr)
        fv = p.factor_var[p.term_ptr[:-1]]
        keep[(deg == 2) & (fv == p.factor_var[p.term_ptr[1:] - 1]) & (fv % 2 == 0)] = False
        return I.Problem(p.n_vars, np.concatenate([[0], np.cumsum(deg[keep])]),
                         np.concatenate([p.factor_var[a:b] for a, b, k in zip(p.term_ptr[:-1], p.term_ptr[1:], keep) if k]),
                         p.coef[keep], p.lower, p.upper)
    if kind == "n1025_wide":       # coefficients past 32 bits: c1 as int64
        return I.dense_quio(1025, -100000, 100000, 100, 100, g)
    if kind == "w1030":            # few variables, wide ranges: three values per thread
        return I.dense_quio(70, -500, 529, 10, 10, g)
    if kind == "w4096":            # four values for every thread of sixteen waves
        return I.dense_quio(65, -2048, 2047, 10, 10, g)
    raise ValueError(kind)


@pytest.mark.parametrize("kind", ["n1030", "n1100_int32", "n1025_wide", "w1030", "w4096"])
@pytest.mark.parametrize("rule", RULES)
def test_against_oracle(kind, rule):
    import torch
    wide_rule = rule in (sa.HEAT_BATH, sa.HEAT_BATH_CLOSED)
    if kind == "n1025_wide" and wide_rule:
        pytest.skip("the oracle enumerates 200001 values per update")
    prob = problem(kind)
    P = oracle.Poly(prob)
    big = prob.n_vars > 1000
    S, reads = (24, 2) if big else (40, 3)
    beta = P.schedule(S)[0]
    beta = np.concatenate([beta[::2], beta[S // 3::-3], beta[1::2]])
    seed = 0xDE45E + rule
    plan = sa.Plan(prob, rule)

    def run(n_reads, z_init=None, s0=0, s1=0, trace=True):
        z = torch.empty((n_reads, prob.n_vars), dtype=torch.int32, device="cuda")
        e = torch.empty(n_reads, dtype=torch.int64, device="cuda")
        h = torch.empty((n_reads, (s1 or len(beta)) - s0), dtype=torch.int64, device="cuda") if trace else None
        zi = None if z_init is None else torch.as_tensor(np.ascontiguousarray(z_init, np.int32), device="cuda")
        plan.run_device(len(beta), n_reads, seed, z, e, beta=beta, stream=torch.cuda.current_stream().cuda_stream,
                        sweep_begin=s0, sweep_end=s1, init_states=zi, trace=h)
        torch.cuda.synchronize()
        return z.cpu().numpy(), e.cpu().numpy(), h.cpu().numpy().view(np.uint64) if trace else None

    z, e, h = run(reads)
    if big or wide_rule:
        assert plan.last_launch()["waves_per_replica"] >= 4
    zo, eo, ho = P.anneal(rule, beta, reads, seed, trace=True)

    def explain(i):
        return parity.localise(P, rule, beta, seed, 0, i, h[i],
                               lambda s, zb: run(i + 1, np.tile(zb, (i + 1, 1)), s, s + 1, False)[0][i])

    parity.check(f"dense team {kind} rule {rule}", reads,
                 lambda i: np.array_equal(z[i], zo[i]) and e[i] == eo[i] and np.array_equal(h[i], ho[i]), explain)
    if not big:
        zt = torch.empty((reads, prob.n_vars), dtype=torch.int32, device="cuda")
        et = torch.empty(reads, dtype=torch.int64, device="cuda")
        sa.anneal_device(prob, rule, len(beta), reads, seed, zt, et, beta=beta, no_alloc=True,
                         stream=torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert np.array_equal(z, zt.cpu().numpy()) and np.array_equal(e, et.cpu().numpy())
    plan.close()
