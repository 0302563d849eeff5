"""GPU parity of the kernels that run the blocks of a hierarchical plan in an
order (colour launches, dataflow with either gather), against the CPU oracle.
Most meshes get an owner plan instead, which has no order; a cell with nine
edges, or a node with seventeen elements, refuses it, so these meshes have one.

Bars: relative L2 1e-12 in binary64 (sums of at most 17 terms of about 60
operations: 1e-14 from rounding at the worst), 1e-6 in binary32 storage against
the oracle's binary32 evaluation (ulp 6e-8 over the same operations)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from meshgen import hex_mesh, quad_mesh  # noqa: E402
from oracle import native  # noqa: E402
from paper_1802_03749_amd import umesh as U  # noqa: E402
from paper_1802_03749_amd.edgeloop import EdgeFluxLoop  # noqa: E402
from paper_1802_03749_amd.hexloop import HexLoop  # noqa: E402


def rel_l2(a, b):
    a = np.asarray(a, np.longdouble); b = np.asarray(b, np.longdouble)
    return float(np.sqrt(((a - b) ** 2).sum()) / np.sqrt((b ** 2).sum()))


def quads_with_hub(nx, ny, seed=6):
    """A quad mesh with five more edges from its middle cell to cells around."""
    m = quad_mesh(nx, ny, seed=seed)
    num = np.argsort(m.cell_nat).reshape(ny, nx)
    i, j = nx // 2, ny // 2
    c = num[j, i]
    far = [num[j + b, i + a] for a, b in ((1, 1), (-1, 1), (1, -1), (-1, -1), (2, 0))]
    m.e2c = np.concatenate([m.e2c, [[c, d] for d in far]]).astype(np.int32)
    m.e2n = np.concatenate([m.e2n, [[m.c2n[c, 0], m.c2n[d, 2]] for d in far]]).astype(np.int32)
    assert np.bincount(m.e2c.ravel()).max() == 9
    return m


def hexes_with_hub(n, seed=6):
    """A hex mesh with nine more elements on the corners of its middle one."""
    m = hex_mesh(n, seed=seed)
    mid = m.e2n[np.argmin(np.abs(m.x[m.e2n].mean(1) - m.x.mean(0)).sum(1))]
    m.e2n = np.concatenate([m.e2n, np.repeat(mid[None], 9, 0)]).astype(np.int32)
    assert np.bincount(m.e2n.ravel()).max() == 17
    return m


def ordered(L, p):
    with pytest.raises(U.UmeshError) as e:
        L.export(p, U.UM_EXP_OWNER_RECORDS)
    return e.value.status == U.UM_ERR_STATE


@pytest.mark.parametrize("schedule,gather,sum_first,layout", [
    (*form, layout) for layout in ("aos", "soa") for form in (
        ("colour_launches", "registers", "auto"), ("dataflow", "registers", "always"),
        ("dataflow", "registers", "never"), ("dataflow", "lds_dma", "always"),
        ("dataflow", "lds_dma", "never"))
    if layout == "aos" or form[1] != "lds_dma"])  # the LDS-DMA gather reads AoS records
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("nx,ny,S", [(47, 33, 128), (9, 7, 512), (150, 90, 512)])
def test_edge_kernels(nx, ny, S, layout, dtype, schedule, gather, sum_first):
    """Every form of the ordered edge kernels: edges per lane, rounds of thread
    colours or LDS atomics, colour groups of whole wavefronts, XCD groups, id
    lists; rounds repeat bit for bit, and XCD groups leave them as they are."""
    m = quads_with_hub(nx, ny)
    L = EdgeFluxLoop(m.x, m.q, m.adt, m.e2n, m.e2c, device=0, layout=layout, dtype=dtype,
                     block_size=S, point_reorder=2)
    ref, bar = (native.edge_loop(m.e2n, m.e2c, m.x, m.q, m.adt), 1e-12) if dtype == "f64" else \
        (native.edge_loop_f32(m.e2n, m.e2c, m.x, m.q, m.adt)[0], 1e-6)

    def sweep(p):
        assert ordered(L, p)
        L.zero_res()
        L.run(p)
        torch.cuda.synchronize()
        r = L.res_user()
        assert rel_l2(r, ref) <= bar
        return r

    base = dict(schedule=schedule, gather=gather, sum_first=sum_first, block_colouring="recolour")
    for ept in (1, 2):
        for kw in (dict(tcmode="lds_atomic"), dict(wave_colour_groups=True),
                   dict(explicit_lists=True)):
            sweep(L.plan("hier", S, elems_per_thread=ept, **base, **kw))
        p = L.plan("hier", S, elems_per_thread=ept, **base)
        assert p.stats["n_launches"] == (1 if schedule == "dataflow" else
                                         p.stats["n_block_colours"])
        rounds = sweep(p)
        assert np.array_equal(rounds, sweep(p))
        assert np.array_equal(rounds, sweep(L.plan("hier", S, elems_per_thread=ept, xcd_groups=8,
                                                   **base)))
    L.close()


@pytest.mark.parametrize("schedule", ["colour_launches", "dataflow"])
@pytest.mark.parametrize("tcmode", ["barrier", "lds_atomic"])
@pytest.mark.parametrize("layout", ["aos", "soa"])
@pytest.mark.parametrize("n,S", [(17, 64), (17, 256), (24, 512), (3, 128)])
def test_hex_kernels(n, S, layout, tcmode, schedule):
    m = hexes_with_hub(n)
    ref = native.hex_loop(m.e2n, m.x, m.v)
    L = HexLoop(m.x, m.v, m.e2n, device=0, layout=layout, block_size=S, point_reorder=3)
    for kw in (dict(), dict(explicit_lists=True), dict(xcd_groups=8)):
        p = L.plan("hier", S, schedule=schedule, tcmode=tcmode, block_colouring="min", **kw)
        assert ordered(L, p)
        L.zero_force()
        L.run(p)
        torch.cuda.synchronize()
        assert rel_l2(L.force_user(), ref) <= 1e-12
    L.close()
