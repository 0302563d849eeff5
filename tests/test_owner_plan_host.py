"""Host-side checks of the owner kernel's plans (no GPU): decoded from the
exported records, every staged position is in range, every cell with an
interior edge is owned by exactly one block, and an owned cell's sides are
exactly the edges around it, with the normals pointing out."""
import numpy as np
import pytest

from meshgen import hex_mesh, quad_mesh
from paper_1802_03749_amd import umesh as U
from paper_1802_03749_amd.edgeloop import EdgeFluxLoop
from paper_1802_03749_amd.hexloop import HexLoop
from paper_1802_03749_amd.timestep import TimeStep2D


def tiles(m, tx, ty):
    nat = m.cell_nat[m.e2c[:, 1]]
    i, j = nat % m.nx, nat // m.nx
    return ((j // ty) * ((m.nx + tx - 1) // tx) + i // tx).astype(np.int32)


def decode(L, p):
    """Per owned cell, in plan order: (cell, [(neighbour, a, b), ...])."""
    rec = L.export(p, U.UM_EXP_OWNER_RECORDS).reshape(-1, 10)
    ids = L.export(p, U.UM_EXP_OWNER_IDS).reshape(rec.shape[0], -1)
    rows = int(rec[:, 1].sum())
    sides = L.export(p, U.UM_EXP_OWNER_SIDES).reshape(rows, -1, 4)
    out, row = [], 0
    for r, it in zip(rec, ids):
        word_off, n_own, nc, nn, c0, c_run, n0, n_run, node_item, n_items = r
        assert word_off == row and c_run <= n_own <= nc <= 1023 and n_run <= nn <= 1023
        assert node_item % 64 == 0 and node_item >= nc - c_run
        assert n_items == node_item + nn - n_run <= ids.shape[1]
        cells = np.concatenate([np.arange(c0, c0 + c_run), it[:nc - c_run]])
        nodes = np.concatenate([np.arange(n0, n0 + n_run), it[node_item:n_items]])
        assert cells.size == np.unique(cells).size == nc
        assert nodes.size == np.unique(nodes).size == nn
        assert nc == 0 or (cells.min() >= 0 and cells.max() < L.C)
        assert nn == 0 or (nodes.min() >= 0 and nodes.max() < L.N)
        for i in range(n_own):
            s = sides[row + i]
            s = s[s[:, 0] >= 0]
            assert s.min(initial=0) >= 0
            assert s[:, 0].max(initial=0) < nc and s[:, 1:3].max(initial=0) < nn
            out.append((int(cells[i]), sorted((int(cells[h]), int(nodes[a]), int(nodes[b]), int(t))
                                              for h, a, b, t in s)))
        row += n_own
    assert row == rows
    return out


@pytest.mark.parametrize("points", [0, 1, 2])
@pytest.mark.parametrize("order,S,layout,explicit", [
    ("rcm+partition", 512, "aos", False), ("partition", 64, "soa", False),
    ("rcm+user", 256, "aos", False), ("rcm", 100, "aos", True), ("none", 256, "soa", False),
    ("rcm+partition", 128, "aos", True)])
@pytest.mark.parametrize("nx,ny", [(61, 37), (5, 3), (2, 1)])
def test_owned_cells_and_their_sides(nx, ny, order, S, layout, explicit, points):
    m = quad_mesh(nx, ny, seed=4)
    L = EdgeFluxLoop(m.x, m.q, m.adt, m.e2n, m.e2c, device=-1, order=order, block_size=S,
                     point_reorder=points, layout=layout, edge_blocks=tiles(m, 16, 8))
    p = L.plan("hier", S, schedule="dataflow", elems_per_thread=2, explicit_lists=explicit,
               gather="lds_dma" if layout == "aos" else "registers")
    e2c, e2n = L.current_map("e2c"), L.current_map("e2n")
    want = {}
    for (l, r), (a, b) in zip(e2c.tolist(), e2n.tolist()):
        want.setdefault(l, []).append((r, a, b, 0))
        want.setdefault(r, []).append((l, b, a, 1))
    try:
        got = decode(L, p)
    except U.UmeshError as e:
        # a random order spreads a block over more cells than it may stage
        assert e.status == U.UM_ERR_STATE and order == "none"
        return
    assert len(got) == len(want) and dict(got) == {c: sorted(s) for c, s in want.items()}
    # a plan of colour launches owns the same cells
    q = L.plan("hier", S, explicit_lists=explicit)
    assert q.stats["n_launches"] == 1 and decode(L, q) == got
    L.close()


def test_edge_between_a_cell_and_itself():
    """Both slots of such an edge are sides of the cell, with opposite
    normals."""
    e2c = np.array([[0, 1], [1, 1]], np.int32)
    e2n = np.array([[0, 1], [2, 3]], np.int32)
    L = EdgeFluxLoop(np.random.default_rng(0).uniform(size=(4, 2)), np.ones((2, 4)), np.ones(2),
                     e2n, e2c, device=-1, order="none")
    p = L.plan("hier", 64, schedule="dataflow", gather="lds_dma")
    assert dict(decode(L, p)) == {0: [(1, 0, 1, 0)], 1: [(0, 1, 0, 1), (1, 2, 3, 0), (1, 3, 2, 1)]}
    L.close()


def test_plans_without_an_owner_kernel():
    """The register gather of a dataflow plan on AoS data, staging of the
    increments only and cells with more than eight sides keep their kernels."""
    m = quad_mesh(30, 20, seed=1)
    L = EdgeFluxLoop(m.x, m.q, m.adt, m.e2n, m.e2c, device=-1)
    for kw in (dict(schedule="dataflow"), dict(staging="inc"), dict(lds_limit_bytes=8192)):
        p = L.plan("hier", 512, **kw)
        with pytest.raises(U.UmeshError):
            L.export(p, U.UM_EXP_OWNER_RECORDS)
        assert p.stats["n_launches"] == (1 if "schedule" in kw else p.stats["n_block_colours"])
    L.close()
    for arms, owned in ((8, True), (9, False)):
        # a star: one cell with `arms` neighbours
        e2c = np.stack([np.zeros(arms, np.int32), np.arange(1, arms + 1, dtype=np.int32)], 1)
        x = np.random.default_rng(0).uniform(size=(2 * arms, 2))
        L = EdgeFluxLoop(x, np.ones((arms + 1, 4)), np.ones(arms + 1),
                         np.arange(2 * arms, dtype=np.int32).reshape(-1, 2), e2c, device=-1,
                         order="none")
        p = L.plan("hier", 64, schedule="dataflow", gather="lds_dma")
        if owned:
            assert sorted(len(s) for _, s in decode(L, p)) == [1] * arms + [arms]
        else:
            with pytest.raises(U.UmeshError):
                L.export(p, U.UM_EXP_OWNER_RECORDS)
        L.close()


@pytest.mark.parametrize("points", [0, 1, 3])
@pytest.mark.parametrize("n,S,explicit", [(9, 256, False), (9, 64, True), (1, 64, False),
                                          (12, 512, False), (2, 128, False)])
def test_hex_owned_nodes_and_their_elements(n, S, explicit, points):
    """Every node is owned once; its sum has one place for each element
    around it, filled by that element's corner at the node."""
    m = hex_mesh(n, seed=3)
    L = HexLoop(m.x, m.v, m.e2n, device=-1, order="rcm+partition", block_size=S,
                point_reorder=points)
    p = L.plan("hier", S, schedule="dataflow", block_colouring="min", explicit_lists=explicit)
    rec = L.export(p, U.UM_EXP_OWNER_RECORDS).reshape(-1, 10)
    ids = L.export(p, U.UM_EXP_OWNER_IDS).reshape(rec.shape[0], -1)
    ex = L.export(p, U.UM_EXP_OWNER_SIDES)
    rows = int(rec[:, 3].sum())
    corners, counts = ex[:16 * rows].reshape(rows, 8, 2), ex[16 * rows:]
    e2n = L.current_map()
    want = [[] for _ in range(L.N)]
    for e, row in enumerate(e2n.tolist()):
        for a, t in enumerate(row):
            want[t].append((tuple(row), a))
    seen, row, at = np.zeros(L.N, int), 0, 0
    for (word_off, n_own, nn, ne, c0, c_run, _, _, _, n_items), it in zip(rec, ids):
        assert word_off == row and c_run <= n_own <= nn <= 1023 and ne <= 1024
        nodes = np.concatenate([np.arange(c0, c0 + c_run), it[:n_items]])
        assert nodes.size == np.unique(nodes).size == nn
        assert nn == 0 or (nodes.min() >= 0 and nodes.max() < L.N)
        w = corners[row:row + ne]
        assert w[:, :, 0].max(initial=0) < max(nn, 1)
        places = [dict() for _ in range(n_own)]
        for el in w:
            for a, (t, place) in enumerate(el):
                if t < n_own:
                    assert place not in places[t]
                    places[t][place] = (tuple(nodes[el[:, 0]].tolist()), a)
        for t in range(n_own):
            k = counts[at + t]
            assert sorted(places[t]) == list(range(k))
            assert sorted(places[t].values()) == sorted(want[nodes[t]])
            seen[nodes[t]] += 1
        row += ne
        at += n_own
    assert row == rows and at == counts.size and np.all(seen == 1)
    L.close()


def step(m, fuse=False, **kw):
    T = TimeStep2D(m.x, m.q, m.e2n, m.e2c, m.b2n, m.b2c, m.c2n, [1.0, 0.35, 0.05, 2.7],
                   device=-1, block_size=64, **kw)
    T.build_plans(flux_block_size=64, schedule="dataflow", gather="lds_dma", elems_per_thread=2,
                  fuse_adt=fuse)
    return T


@pytest.mark.parametrize("fuse", [False, True])
@pytest.mark.parametrize("points", [0, 2])
@pytest.mark.parametrize("nx,ny", [(23, 17), (2, 1), (5, 1)])
def test_step_plan_has_every_side_of_every_cell(nx, ny, points, fuse):
    """The step's plan owns every cell; side k of a cell runs from node k to
    node k + 1 of its row and has the edge or boundary edge that lies there.
    Steps that evaluate adt first have the corners of the other staged cells."""
    m = quad_mesh(nx, ny, seed=8)
    T = step(m, fuse, point_reorder=points)
    h = T._whole.handle
    get = lambda f: (lambda out: (U.um_plan_export(h, f, out, out.size), out)[1])(
        np.empty(U.um_plan_export(h, f), np.int32))
    table = lambda mp, k: (lambda out: (U.um_get_map(T.ctx, mp, out), out)[1])(
        np.empty((k, {T.m_c2n: 4, T.m_b2c: 1}.get(mp, 2)), np.int32))
    rec = get(U.UM_EXP_OWNER_RECORDS).reshape(-1, 10)
    ids = get(U.UM_EXP_OWNER_IDS).reshape(rec.shape[0], -1)
    sides = get(U.UM_EXP_OWNER_SIDES).reshape(-1, 4, 4)
    c2n = table(T.m_c2n, T.C)
    out = {}  # (cell, a, b) -> neighbour
    for (l, r), (a, b) in zip(table(T.m_e2c, T.E).tolist(), table(T.m_e2n, T.E).tolist()):
        out[l, a, b] = (r, 0)
        out[r, b, a] = (l, 1)
    for (c,), (a, b) in zip(table(T.m_b2c, T.B).tolist(), table(T.m_b2n, T.B).tolist()):
        out[c, a, b] = (-2, 0)
    seen, row = [], 0
    for (_, n_own, nc, nn, c0, c_run, n0, n_run, node_item, n_items), it in zip(rec, ids):
        assert c_run <= n_own <= nc <= 1022 and nn <= 1022
        cells = np.concatenate([np.arange(c0, c0 + c_run), it[:nc - c_run]])
        nodes = np.concatenate([np.arange(n0, n0 + n_run), it[node_item:n_items]])
        for i in range(n_own):
            c = int(cells[i])
            seen.append(c)
            for k in range(4):
                h, a, b, slot = sides[row + i, k]
                want = out[c, int(c2n[c, k]), int(c2n[c, (k + 1) % 4])]
                assert (nodes[a], nodes[b]) == (c2n[c, k], c2n[c, (k + 1) % 4])
                assert ((int(cells[h]) if h >= 0 else int(h)), int(slot)) == want
        row += n_own
        for i in range(n_own, 0 if fuse else nc):
            lo, hi = it[n_items + 2 * (i - n_own):][:2]
            corners = [(lo >> 10) & 1023, (lo >> 20) & 1023, hi & 1023, (hi >> 10) & 1023]
            assert nodes[corners].tolist() == c2n[cells[i]].tolist()
    assert sorted(seen) == list(range(T.C))
    assert T.step_launches() == 2
    T.close()


def test_step_plan_refused():
    """A boundary edge that runs the other way round, a second one on the same
    side, an edge between nodes that no side joins, and a cell without an
    edge: the loops run separately."""
    m = quad_mesh(6, 5, seed=8)
    m.b2n[3] = m.b2n[3, ::-1]
    T = step(m)
    assert T._whole is None and T.step_launches() > 2
    T.close()
    m = quad_mesh(6, 5, seed=8)
    m.b2n, m.b2c = np.concatenate([m.b2n, m.b2n[:1]]), np.concatenate([m.b2c, m.b2c[:1]])
    assert step(m)._whole is None
    m = quad_mesh(6, 5, seed=8)
    m.e2n[7, 0] = m.e2n[8, 1]
    assert step(m)._whole is None
    assert step(quad_mesh(1, 1, seed=8))._whole is None
