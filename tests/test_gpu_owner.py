"""GPU parity of the owner kernels (blocks without an order) against the
CPU oracle, at the forms their plans take.  Edge loop: cells whose sides close
a ring and cells of any other shape with up to eight sides, runs and listed
ids, both layouts and storage types, one and many wavefronts per block.  Hex
loop: grids at several block sizes and nodes with up to sixteen elements.

Bars: relative L2 1e-12 in binary64 (sums of at most 8 fluxes of about 30
operations: 1e-15 from rounding), 1e-6 in binary32 storage against the
oracle's binary32 evaluation (ulp 6e-8 over the same operations)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from meshgen import hex_mesh, quad_mesh  # noqa: E402
from oracle import native  # noqa: E402
from paper_1802_03749_amd import umesh as U  # noqa: E402
from paper_1802_03749_amd.edgeloop import EdgeFluxLoop  # noqa: E402
from paper_1802_03749_amd.hexloop import HexLoop  # noqa: E402
from paper_1802_03749_amd.timestep import TimeStep2D  # noqa: E402


def rel_l2(a, b):
    a = np.asarray(a, np.longdouble); b = np.asarray(b, np.longdouble)
    return float(np.sqrt(((a - b) ** 2).sum()) / np.sqrt((b ** 2).sum()))


def random_cells(C, sides, seed):
    """C cells of at most `sides` sides joined at random: no rings."""
    rng = np.random.default_rng(seed)
    ends = rng.permutation(np.repeat(np.arange(C), sides))[:C * sides // 2 * 2].reshape(-1, 2)
    e2c = ends[ends[:, 0] != ends[:, 1]].astype(np.int32)
    N = 3 * C
    rho, p = rng.uniform(0.9, 1.1, C), rng.uniform(0.9, 1.1, C)
    u, v = rng.uniform(-0.2, 0.2, (2, C))
    q = np.stack([rho, rho * u, rho * v, p / 0.4 + 0.5 * rho * (u * u + v * v)], 1)
    return (rng.uniform(-1, 1, (N, 2)), q, rng.uniform(1, 2, C),
            rng.integers(0, N, e2c.shape).astype(np.int32), e2c)


def check(mesh, dtype, layout, **kw):
    x, q, adt, e2n, e2c = mesh
    L = EdgeFluxLoop(x, q, adt, e2n, e2c, device=0, layout=layout, dtype=dtype, **kw.pop("loop"))
    S = L.part_block_size or kw.pop("S")
    for flow in (False, True):  # one sweep each
        p = L.plan("hier", S, **(dict(schedule="dataflow", elems_per_thread=2,
                                      gather="lds_dma" if layout == "aos" else "registers")
                                 if flow else {}), **kw)
        assert p.stats["n_launches"] == 1 and L.export(p, U.UM_EXP_OWNER_RECORDS).size
        L.run(p)
    sides = L.export(p, U.UM_EXP_OWNER_SIDES)
    torch.cuda.synchronize()
    if dtype == "f64":
        assert rel_l2(L.res_user(), 2 * native.edge_loop(e2n, e2c, x, q, adt)) <= 1e-12
    else:
        r32, _ = native.edge_loop_f32(e2n, e2c, x, q, adt)
        assert rel_l2(L.res_user(), 2 * r32) <= 1e-6
    n = int(L.export(p, U.UM_EXP_OWNER_RECORDS).reshape(-1, 10)[:, 1].sum())
    L.close()
    return sides.size // (4 * n)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("layout", ["aos", "soa"])
@pytest.mark.parametrize("nx,ny,S,points,explicit", [
    (130, 67, 64, 2, False), (130, 67, 512, 0, False), (63, 64, 1024, 1, True),
    (2, 1, 64, 2, False), (9, 200, 256, 3, False)])
def test_ring_cells(nx, ny, S, points, explicit, layout, dtype):
    m = quad_mesh(nx, ny, seed=6)
    assert check((m.x, m.q, m.adt, m.e2n, m.e2c), dtype, layout, explicit_lists=explicit,
                 loop=dict(order="rcm+partition", block_size=S, point_reorder=points)) == 4


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("layout", ["aos", "soa"])
@pytest.mark.parametrize("sides", [3, 4, 5, 8])
def test_other_cells(sides, layout, dtype):
    mesh = random_cells(90, sides, seed=sides)
    assert check(mesh, dtype, layout, S=64, loop=dict(order="none")) == (4 if sides <= 4 else 8)


def check_hex(x, v, e2n, layout, loop, S, **kw):
    L = HexLoop(x, v, e2n, device=0, layout=layout, **loop)
    for schedule in ("dataflow", "colour_launches"):  # one sweep each
        p = L.plan("hier", S, schedule=schedule, block_colouring="recolour", **kw)
        assert p.stats["n_launches"] == 1 and L.export(p, U.UM_EXP_OWNER_RECORDS).size
        L.run(p)
    torch.cuda.synchronize()
    assert rel_l2(L.force_user(), 2 * native.hex_loop(e2n, x, v)) <= 1e-12
    L.close()


@pytest.mark.parametrize("layout", ["aos", "soa"])
@pytest.mark.parametrize("n,S,points,explicit", [(1, 64, 1, False), (9, 64, 3, False),
                                                 (17, 256, 2, False), (17, 256, 0, True),
                                                 (16, 512, 3, False), (23, 128, 1, False)])
def test_hex(n, S, points, explicit, layout):
    m = hex_mesh(n, seed=6)
    check_hex(m.x, m.v, m.e2n, layout, dict(order="rcm+partition", block_size=S,
                                            point_reorder=points), S, explicit_lists=explicit,
              tcmode="lds_atomic" if n == 23 else "barrier")


@pytest.mark.parametrize("layout", ["aos", "soa"])
@pytest.mark.parametrize("around", [3, 9, 16])
def test_hex_nodes_of_other_degrees(around, layout):
    """Elements on random nodes, up to 16 around a node."""
    rng = np.random.default_rng(around)
    N = 160
    e2n = rng.permutation(np.repeat(np.arange(N), around))[:N * around // 8 * 8]
    e2n = e2n.reshape(-1, 8).astype(np.int32)
    check_hex(rng.uniform(-1, 1, (N, 3)), rng.uniform(-1, 1, (N, 3)), e2n, layout,
              dict(order="none"), 64)


def test_non_finite_states_stay_with_their_neighbours():
    """An infinite or NaN state reaches the residuals of its own cell and of
    the cells around it, as in the waiting kernel, and no other."""
    m = quad_mesh(40, 30, seed=2)
    q = m.q.copy()
    q[100, 3], q[500, 1] = np.inf, np.nan
    out = []
    for gather in ("lds_dma", "registers"):
        L = EdgeFluxLoop(m.x, q, m.adt, m.e2n, m.e2c, device=0, block_size=128)
        L.run(L.plan("hier", 128, schedule="dataflow", gather=gather))
        torch.cuda.synchronize()
        out.append(L.res_user())
        L.close()
    assert np.array_equal(np.isfinite(out[0]), np.isfinite(out[1]))
    fine = np.isfinite(out[0])
    assert 0 < (~fine).sum() <= 40 and rel_l2(out[0][fine], out[1][fine]) <= 1e-12


QINF = np.array([1.0, 0.35, 0.05, 2.7])


@pytest.mark.parametrize("opts", [dict(schedule="dataflow", gather="lds_dma", elems_per_thread=2),
                                  dict()], ids=["dataflow", "default"])
@pytest.mark.parametrize("fuse", [True, False])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("nx,ny,S,points", [(150, 70, 512, 2), (37, 53, 64, 0), (2, 1, 64, 1),
                                            (61, 260, 1024, 2)])
def test_whole_step(nx, ny, S, points, dtype, fuse, opts):
    """Edge flux, boundary flux and update as one loop against the separate
    loops from the same state: two steps, the first with residuals that hold
    something.  Bars: binary64 1e-12; binary32 q and adt 4 ulp of 6e-8."""
    m = quad_mesh(nx, ny, seed=11)
    start = np.random.default_rng(1).uniform(-1e-2, 1e-2, (nx * ny, 4))
    T = []
    for whole in (True, False):
        t = TimeStep2D(m.x, m.q, m.e2n, m.e2c, m.b2n, m.b2c, m.c2n, QINF, device=0, block_size=S,
                       point_reorder=points, dtype=dtype)
        t.build_plans(flux_block_size=S, fuse_adt=fuse, **opts)
        assert t._whole is not None
        if not whole:
            t._whole = None
        t.res.copy_(torch.from_numpy(start))
        T.append(t)
    for k in (1, 2):
        for t in T:
            t.step()
        torch.cuda.synchronize()
        a, b = T
        bar = 1e-12 if dtype == "f64" else 2.4e-7
        assert rel_l2(a.q_user(), b.q_user()) <= bar
        assert rel_l2(a.adt_user(), b.adt_user()) <= bar
        assert not a.res.view(torch.int64).any() and not b.res.any()
        assert abs(a.rms.item() - b.rms.item()) <= (1e-12 if dtype == "f64" else 1e-6) * b.rms.item()
    for t in T:
        t.close()


def test_whole_step_refuses_overlapping_dats():
    """res re-pointed into q is refused at the step, as by the edge flux loop."""
    m = quad_mesh(20, 10, seed=3)
    t = TimeStep2D(m.x, m.q, m.e2n, m.e2c, m.b2n, m.b2c, m.c2n, QINF, device=0, block_size=64)
    t.build_plans(flux_block_size=64)
    assert t._whole is not None
    U.um_set_dat_ptr(t.ctx, t.d_res, t.q.data_ptr())
    with pytest.raises(U.UmeshError) as ei:
        t.step()
    assert ei.value.status == U.UM_ERR_ARG
    t.close()


def test_whole_step_in_a_graph():
    """Replays of a captured step against eager steps."""
    m = quad_mesh(200, 90, seed=12)
    T = [TimeStep2D(m.x, m.q, m.e2n, m.e2c, m.b2n, m.b2c, m.c2n, QINF, device=0,
                    block_size=256) for _ in range(2)]
    for t in T:
        t.build_plans(flux_block_size=256, schedule="dataflow", gather="lds_dma",
                      elems_per_thread=2, fuse_adt=True)
        t.step()
    g = U.HipGraph(T[0].step)
    for k in range(4):
        g.replay()
        T[1].step()
        torch.cuda.synchronize()
        assert torch.equal(T[0].q, T[1].q) and torch.equal(T[0].adt, T[1].adt)
        assert T[0].rms.item() == T[1].rms.item()
    g.close()
    for t in T:
        t.close()
