"""GPU: the heat bath's draws at the edges of their ranges against the oracle, sweep by sweep, at
tests/parity.py's bar: widths around a wavefront, its multiples and the forms' limits, slopes of both
signs, flat and steep, from beta = 0 to frozen."""
import numpy as np
import pytest

import oracle
from paper_2511_17245_amd import inputs as I
from paper_2511_17245_amd import sa
from tests import parity

pytestmark = pytest.mark.gpu


def run(prob, beta, reads, seed, G, z_init=None, s0=0, s1=0, trace=True):
    plan = sa.Plan(prob, sa.HEAT_BATH)
    out = plan.run(len(beta), reads, seed, beta=beta, waves_per_replica=G, lanes_per_update=64,
                   init_states=z_init, sweep_begin=s0, sweep_end=s1, trace=trace)
    plan.close()
    return out


def check(name, prob, beta, reads, seed, G):
    P = oracle.Poly(prob)
    zo, eo, ho = P.anneal(sa.HEAT_BATH, beta, reads, seed, trace=True)
    z, e, h = run(prob, beta, reads, seed, G)

    def explain(i):
        def after(s, zb):
            return run(prob, beta, i + 1, seed, G, np.tile(zb, (i + 1, 1)), s, s + 1, trace=False)[0][i]
        return parity.localise(P, sa.HEAT_BATH, beta, seed, 0, i, h[i], after)

    parity.check(name, reads,
                 lambda i: np.array_equal(z[i], zo[i]) and e[i] == eo[i] and np.array_equal(h[i], ho[i]), explain)


def betas(scale):
    """0, so small that every weight is 1, then from flat to frozen for energy differences of `scale`."""
    return np.concatenate([[0.0, 1e-300, 1e-20 / scale], np.geomspace(1e-4, 1e4, 17) / scale])


@pytest.mark.parametrize("width", [2, 63, 64, 65, 512, 513, 2049, 65536, 65537, (1 << 20) + 3])
def test_linear(width):
    """No variable to a power above one: the inverse of the distribution, in each of its precisions."""
    lo = -(width // 3)
    prob = I.multilinear(9, 3, 2)
    prob.lower[:] = lo
    prob.upper[:] = lo + width - 1
    for G in (1, 2):
        check(f"linear W {width} G {G}", prob, betas(float(width) ** 3), 2 if width > 4096 else 8, 91 + width, G)


@pytest.mark.parametrize("width", [2, 63, 64, 65, 511, 512, 513, 2048, 2049])
@pytest.mark.parametrize("kind", ["squares", "dense", "powers"])
def test_powers(width, kind):
    """Powers above one: single precision up to 512 values, double beyond; minima inside the range, at an
    end and (negative squares) at both."""
    g = np.random.Generator(np.random.PCG64(width))
    lo = -(width // 3)
    scale = float(width) ** 2 * 10
    if kind == "squares":
        prob = I.erdos_renyi_quio(12, 3.0, lo, lo + width - 1, 10, 20, g)
        terms = [(int(c), [i, i]) for i, c in enumerate(g.integers(-6, 7, 12))]
        prob = I.from_terms(12, terms + [(3, [0, 1]), (-2, [1, 2]), (5, [3]), (-7, [4])], prob.lower, prob.upper)
    elif kind == "dense":
        prob = I.dense_quio(12, lo, lo + width - 1, 10, 10, g)
    else:
        prob = I.random_huio(12, 40, [1, 2, 3], lo, lo + width - 1, 5, g)
        scale *= width
    for G in (1, 2):
        if kind == "dense" and G == 2:
            continue
        check(f"{kind} W {width} G {G}", prob, betas(scale), 8, 17 + width, G)


def test_single_precision_over_many_draws():
    """Enough draws that thousands of them pass near a step of the distribution."""
    g = np.random.Generator(np.random.PCG64(5))
    prob = I.dense_quio(30, -100, 100, 10, 10, g)
    check("many draws", prob, np.geomspace(1e-5, 1e-1, 120), 400, 3, 1)
