"""GPU: what the options ask for is what runs."""
import numpy as np
import pytest

from paper_2511_17245_amd import inputs as I
from paper_2511_17245_amd import sa

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rule", [sa.METROPOLIS, sa.HEAT_BATH])
def test_lanes_64_is_one_wavefront_per_update(rule):
    """A dense problem that goes to a team of waves by itself stays with one wavefront per update when that
    is asked for; the results are the same."""
    prob = I.dense_quio(1030, -3, 5, 10, 10, np.random.Generator(np.random.PCG64(4)))
    plan = sa.Plan(prob, rule)
    z, e = plan.run(6, 2, 99)
    assert plan.last_launch()["kernel_variant"] // 1000000 == 3 and plan.last_launch()["waves_per_replica"] > 1
    z64, e64 = plan.run(6, 2, 99, lanes_per_update=64)
    assert plan.last_launch()["kernel_variant"] < 1000000 and plan.last_launch()["waves_per_replica"] == 1
    assert np.array_equal(z, z64) and np.array_equal(e, e64)
    plan.close()


def test_autotune_is_for_the_persistent_kernel():
    """A batch whose problems all go to the lane kernel has nothing to tune, and leaves no choice behind for a
    batch of the same size that has."""
    g = np.random.Generator(np.random.PCG64(9))
    probs = [I.erdos_renyi_quio(600 + i, 4.0, -7, 8, 10, 10, g) for i in range(3)]
    def batch(rule):
        items = [I.Workload(p, rule, 40, 8, 3 + i, i) for i, p in enumerate(probs)]
        b = sa.Batch(items, autotune=True)
        info = b.info()
        b.run()
        got = b.results()
        b.close()
        for w, (z, e) in zip(items, got):
            plan = sa.Plan(w.problem, rule)
            zp, ep = plan.run(w.n_sweeps, w.n_reads, w.seed, instance_id=w.instance_id)[:2]
            plan.close()
            assert np.array_equal(z, zp) and np.array_equal(e, ep)
        return info["tune_ms"]
    assert batch(sa.HEAT_BATH) == 0.0
    assert batch(sa.METROPOLIS) > 0.0
    assert batch(sa.METROPOLIS) == 0.0   # (chosen before)
