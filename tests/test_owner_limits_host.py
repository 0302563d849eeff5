"""The largest blocks that the owner kernels take: 1022 staged points of a set
(10-bit positions, of which one means no cell and one the far field), 1024
evaluated elements (lanes of a workgroup).  Host-only contexts."""
import numpy as np
import pytest

from paper_1802_03749_amd import umesh as U
from paper_1802_03749_amd.edgeloop import EdgeFluxLoop
from paper_1802_03749_amd.hexloop import HexLoop


def records(L, p):
    """The plan's owner records, None if it is not an owner plan."""
    try:
        return L.export(p, U.UM_EXP_OWNER_RECORDS).reshape(-1, 10)
    except U.UmeshError as e:
        assert e.status == U.UM_ERR_STATE
        return None


@pytest.mark.parametrize("schedule", ["colour_launches", "dataflow"])
@pytest.mark.parametrize("cells,nodes", [(1022, 7), (1023, 7), (521, 1022), (521, 1023),
                                         (1022, 1022)])
def test_staged_cells_and_nodes(cells, nodes, schedule):
    """A chain of cells in one block, its edges over the given nodes."""
    e2c = np.stack([np.arange(cells - 1), np.arange(1, cells)], 1)
    slots = np.arange(2 * (cells - 1)) % nodes
    L = EdgeFluxLoop(np.zeros((nodes, 2)), np.ones((cells, 4)), np.ones(cells),
                     slots.reshape(-1, 2), e2c, device=-1, order="none")
    kw = dict(schedule=schedule, gather="lds_dma") if schedule == "dataflow" else {}
    r = records(L, L.plan("hier", 1024, lds_limit_bytes=163840, **kw))
    if max(cells, nodes) <= 1022:
        assert r[:, 2].tolist() == [cells] and r[:, 3].tolist() == [nodes]
    else:
        assert r is None
    L.close()


@pytest.mark.parametrize("schedule", ["colour_launches", "dataflow"])
@pytest.mark.parametrize("nodes", [1022, 1023])
def test_staged_nodes_of_hexes(nodes, schedule):
    e2n = (np.arange(1024) % nodes).reshape(-1, 8)
    L = HexLoop(np.zeros((nodes, 3)), np.zeros((nodes, 3)), e2n, device=-1, order="none")
    r = records(L, L.plan("hier", 128, schedule=schedule, lds_limit_bytes=163840))
    assert r is None if nodes > 1022 else r[:, 2].tolist() == [nodes]
    L.close()


@pytest.mark.parametrize("elements", [1024, 1025])
def test_evaluated_hexes(elements):
    """Groups of at most sixteen elements on the same eight nodes; the 1025th
    element lies in the second block, around nodes of the first."""
    group = np.arange(elements) % 65
    e2n = 8 * group[:, None] + np.arange(8)
    L = HexLoop(np.zeros((520, 3)), np.zeros((520, 3)), e2n, device=-1, order="none")
    r = records(L, L.plan("hier", 1024, lds_limit_bytes=163840))
    assert r is None if elements > 1024 else r[:, 3].tolist() == [1024]
    L.close()
