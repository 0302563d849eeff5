"""The autotuner's choice among owner plans over the same blocks: by the timer
where launch order or id lists differ; for binary32 AoS edge loops the
dataflow rounding of one kernel's two."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from meshgen import quad_mesh  # noqa: E402
from paper_1802_03749_amd import umesh as U  # noqa: E402
from paper_1802_03749_amd.edgeloop import PARAMS, EdgeFluxLoop  # noqa: E402


def tune(L, candidates, reps):
    opts = []
    for c in candidates:
        o = U.um_plan_opts()
        o.strategy, o.block_size, o.elems_per_thread = U.UM_STRAT_HIER, 512, 1
        o.block_colouring = U.UM_BCOL_RECOLOUR
        for k, v in c.items():
            setattr(o, k, v)
        opts.append(o)
    h, best, ms = U.um_plan_autotune(L.ctx, U.UM_K_EDGE_FLUX_LF2D, L.args(), L.s_edges, opts,
                                     PARAMS, L.stream, reps)
    assert U.um_plan_export(h, U.UM_EXP_OWNER_RECORDS) > 0
    U.um_plan_destroy(h)
    return best, ms


@pytest.mark.parametrize("reverse", [False, True])
def test_timer_decides_between_launch_orders(reverse):
    """Two XCD groups scatter neighbouring blocks over the XCDs, eight keep
    them together: whichever is listed first, the smaller time wins."""
    m = quad_mesh(1200, 600, seed=1)
    L = EdgeFluxLoop(m.x, m.q, m.adt, m.e2n, m.e2c, device=0, order="rcm+partition",
                     point_reorder=2)
    c = [dict(xcd_groups=2), dict(), dict(explicit_lists=1),
         dict(xcd_groups=2, schedule=U.UM_SCHED_DATAFLOW, gather=U.UM_GATHER_LDS_DMA)]
    best, ms = tune(L, c[::-1] if reverse else c, 30)
    assert ms[best] == min(ms) and min(ms) > 0
    L.close()


@pytest.mark.parametrize("reverse", [False, True])
def test_one_kernel_in_two_roundings(reverse):
    m = quad_mesh(130, 67, seed=6)
    L = EdgeFluxLoop(m.x, m.q, m.adt, m.e2n, m.e2c, device=0, dtype="f32")
    c = [dict(), dict(schedule=U.UM_SCHED_DATAFLOW, gather=U.UM_GATHER_LDS_DMA)]
    best, ms = tune(L, c[::-1] if reverse else c, 3)
    assert best == (0 if reverse else 1) and ms[0] == ms[1] > 0
    L.close()
