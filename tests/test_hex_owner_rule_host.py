"""Which dataflow hex plans run the owner kernel on large meshes: those that
measured faster on it (host-only contexts; the bounds are in elements)."""
import numpy as np
import pytest

from paper_1802_03749_amd import umesh as U
from paper_1802_03749_amd.hexloop import HexLoop


def grid(nx, ny, nz, bricks):
    """Elements of a hex grid row by row, or brick by brick of 8x8x4."""
    k, j, i = (a.ravel() for a in np.meshgrid(*(np.arange(n) for n in (nz, ny, nx)), indexing="ij"))
    if bricks:
        o = np.lexsort((i % 8, j % 8, k % 4, i // 8, j // 8, k // 4))
        i, j, k = i[o], j[o], k[o]
    a, b = nx + 1, (nx + 1) * (ny + 1)
    first = i + a * j + b * k
    corner = np.array([0, 1, a + 1, a, b, b + 1, b + a + 1, b + a])
    return (first[:, None] + corner).astype(np.int32), b * (nz + 1)


@pytest.mark.parametrize("shape,bricks,want", [
    # rows: 64 elements per block evaluate four elements per element
    ((96, 96, 86), False, {("aos", "lds_atomic"): True}),
    ((96, 96, 88), False, {("aos", "lds_atomic"): False, ("aos", "barrier"): True,
                           ("soa", "lds_atomic"): True}),
    ((104, 104, 112), False, {("aos", "barrier"): False, ("soa", "lds_atomic"): False}),
    # bricks: 256 per block, 1.6 elements per element
    ((112, 112, 124), True, {("aos", "lds_atomic"): True}),
    ((112, 112, 128), True, {("aos", "lds_atomic"): False, ("aos", "barrier"): True,
                             ("soa", "lds_atomic"): True}),
])
def test_large_dataflow_plans(shape, bricks, want):
    e2n, nodes = grid(*shape, bricks)
    zero = np.zeros((nodes, 3))
    for layout in ("aos", "soa"):
        modes = [t for (lay, t) in want if lay == layout]
        if not modes:
            continue
        L = HexLoop(zero, zero, e2n, device=-1, order="none", layout=layout)
        for tcmode in modes:
            p = L.plan("hier", 256 if bricks else 64, schedule="dataflow", tcmode=tcmode)
            try:
                owner = U.um_plan_export(p.handle, U.UM_EXP_OWNER_RECORDS) > 0
            except U.UmeshError:
                owner = False
            assert owner == want[layout, tcmode], (layout, tcmode)
        L.close()
