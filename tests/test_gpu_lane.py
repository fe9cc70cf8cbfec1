"""GPU: the lane kernel (heat bath of multilinear pair problems, one update per lane) against the oracle,
sweep by sweep, at tests/parity.py's bar."""
import numpy as np
import pytest

import oracle
from paper_2511_17245_amd import inputs as I
from paper_2511_17245_amd import sa
from tests import parity

pytestmark = pytest.mark.gpu


def problem(kind):
    g = np.random.Generator(np.random.PCG64(4242))
    if kind == "mixed":            # ranges of 1 to 120 values, several chunks per level, ragged
        p = I.erdos_renyi_quio(1501, 6.0, -60, 59, 10, 20, g)
        w = g.integers(1, 121, size=p.n_vars)
        p.lower = (-60 + g.integers(0, 121 - w)).astype(np.int32)
        p.upper = (p.lower + w - 1).astype(np.int32)
        return p
    if kind == "binary":
        return I.erdos_renyi_quio(700, 3.0, 0, 1, 3, 3, g)
    if kind == "wide":             # 2001 values: the single-precision bound decides fewer draws
        return I.erdos_renyi_quio(400, 4.0, -1000, 1000, 10, 20, g)
    if kind == "hub":              # rows of a hundred records, past those loaded ahead; 32-bit records
        terms = [(int(g.integers(-9, 10)) or 1, [i]) for i in range(300)]
        terms += [((1 << 17) * (int(g.integers(-3, 4)) or 1), [0, j]) for j in range(100, 200)]
        terms += [(int(g.integers(-5, 6)) or 1, [i, i + 150]) for i in range(1, 140)]
        return I.from_terms(300, terms, -7, 7)
    if kind == "big":              # coefficients past 32 bits: 64-bit sums
        return I.erdos_renyi_quio(500, 4.0, -3000, 3001, 2000000, 1000, g)
    raise ValueError(kind)


@pytest.mark.parametrize("kind", ["mixed", "binary", "wide", "hub", "big"])
@pytest.mark.parametrize("rule", [sa.HEAT_BATH, sa.HEAT_BATH_CLOSED])
@pytest.mark.parametrize("reads", [3, 600])
def test_against_oracle(kind, rule, reads):
    import torch
    if reads > 3 and kind not in ("mixed", "binary"):
        pytest.skip("many reads (fewer waves each) on two problems")
    prob = problem(kind)
    P = oracle.Poly(prob)
    S = 30 if kind in ("wide", "big") else 60
    S = S if reads == 3 else 20
    beta = P.schedule(S)[0]
    beta[3] = 0.0
    seed = 0x1A4E + rule
    plan = sa.Plan(prob, rule)

    def run(n_reads, z_init=None, s0=0, s1=0, lanes=0):
        z = torch.empty((n_reads, prob.n_vars), dtype=torch.int32, device="cuda")
        e = torch.empty(n_reads, dtype=torch.int64, device="cuda")
        h = torch.empty((n_reads, (s1 or S) - s0), dtype=torch.int64, device="cuda")
        zi = None if z_init is None else torch.as_tensor(np.ascontiguousarray(z_init, np.int32), device="cuda")
        plan.run_device(S, n_reads, seed, z, e, beta=beta, stream=torch.cuda.current_stream().cuda_stream,
                        sweep_begin=s0, sweep_end=s1, init_states=zi, trace=h, lanes_per_update=lanes)
        torch.cuda.synchronize()
        return z.cpu().numpy(), e.cpu().numpy(), h.cpu().numpy().view(np.uint64)

    z, e, h = run(reads)
    assert plan.last_launch()["lanes_per_update"] == 1
    zo, eo, ho = P.anneal(rule, beta, reads, seed, trace=True)

    def explain(i):
        return parity.localise(P, rule, beta, seed, 0, i, h[i],
                               lambda s, zb: run(i + 1, np.tile(zb, (i + 1, 1)), s, s + 1, 64)[0][i])

    parity.check(f"lane {kind} rule {rule} reads {reads}", reads,
                 lambda i: np.array_equal(z[i], zo[i]) and e[i] == eo[i] and np.array_equal(h[i], ho[i]), explain)
    zr, er, _ = run(reads, z_init=run(reads, s1=S - 16)[0], s0=S - 16)   # resumed, 16 sweeps left
    assert np.array_equal(zr, z) and np.array_equal(er, e)
    plan.close()
