"""Timing of a time step's loops through their own plans."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from meshgen import quad_mesh  # noqa: E402
from paper_1802_03749_amd import umesh as U  # noqa: E402
from paper_1802_03749_amd.timestep import TimeStep2D  # noqa: E402


def rel_l2(a, b):
    return float(np.sqrt(((a - b) ** 2).sum() / (b ** 2).sum()))


@pytest.mark.parametrize("fuse", [False, True])
def test_step_records_the_times_of_a_timed_loop(fuse):
    """Steps with and without the timing of a loop: launches recorded for each
    timed step, none for the others, the same state to rounding (binary64,
    four steps: 1e-12)."""
    m = quad_mesh(90, 70, seed=3)
    T = [TimeStep2D(m.x, m.q, m.e2n, m.e2c, m.b2n, m.b2c, m.c2n, [1.0, 0.35, 0.05, 2.7], device=0)
         for _ in range(2)]
    for t in T:
        t.build_plans(fuse_adt=fuse)
    timed = T[0].plans
    for k, on in enumerate((True, False, True, False)):
        for p in timed.values():
            U.um_plan_set_timing(p.handle, on)
        for t in T:
            t.step()
        for name, p in timed.items():
            ms, n = U.um_plan_timing(p.handle)
            runs = on and (name != "adt" or not fuse or k == 0)  # fused: adt before step 0 only
            assert n == (p.stats["n_launches"] if runs else 0) and (ms > 0) == runs, name
    assert rel_l2(T[0].q_user(), T[1].q_user()) <= 1e-12
    assert abs(T[0].rms.item() / T[1].rms.item() - 1) <= 1e-12
    for t in T:
        t.close()
