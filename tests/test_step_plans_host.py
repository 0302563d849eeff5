"""Which loop a time step runs (host-only contexts)."""
import numpy as np
import torch

from meshgen import quad_mesh
from paper_1802_03749_amd import umesh as U
from paper_1802_03749_amd.timestep import TimeStep2D

QINF = np.array([1.0, 0.35, 0.05, 2.7])


def make(m, **kw):
    T = TimeStep2D(m.x, m.q, m.e2n, m.e2c, m.b2n, m.b2c, m.c2n, QINF, device=-1, block_size=64,
                   **kw)
    T.stream, T.res = None, torch.zeros(T.C, 4, dtype=torch.float64)
    return T


def test_timed_loops_run_separately():
    """The loops' own plans record nothing in the step as one loop."""
    T = make(quad_mesh(23, 17, seed=8))
    T.build_plans(flux_block_size=64)
    whole = T.step_launches()
    for p in T.plans.values():
        U.um_plan_set_timing(p.handle, True)
        assert whole == 2 < T.step_launches()
        U.um_plan_set_timing(p.handle, False)
        assert T.step_launches() == whole
    U.um_plan_set_timing(T.plans["flux"].handle, True)
    T.build_plans(flux_block_size=64)  # new plans are not timed
    assert T.step_launches() == whole
    T.close()
