"""Workloads whose speed matters to a user of this package, for a timing harness.

A case is a dict of plain values; `prepare(case, seed)` sets up on the GPU what
a solver keeps between passes (the reordered mesh, its dats, the plan),
`run(state)` makes one pass through the package's public drivers, and
`exact(case, seed)` evaluates the same pass with numpy in binary64.

Four loops are covered:

  edge   one sweep of the 2D edge-flux loop (EdgeFluxLoop.run)
  hex    one sweep of the 3D hexahedral element loop (HexLoop.run)
  step   one explicit time step: adt, edge flux, boundary flux, update
         (TimeStep2D.step)
  batch  one time step of a batch of small meshes as their disjoint union,
         replayed from a captured graph (BatchedSteps)

Meshes are jittered quad or hex grids with random states.  Quad cells and
nodes come numbered along anti-diagonals (the level order a bandwidth-reducing
generator leaves) or row by row.

Where the library renumbers points by its own partition, its results lie in
a numbering that only the library knows, and `exact` has no value for them;
where the points keep the caller's order, or the caller's own blocks decide
the order, it has.
"""
from __future__ import annotations

import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_1802_03749_amd import measure
from paper_1802_03749_amd.batched import BatchedSteps
from paper_1802_03749_amd.edgeloop import EdgeFluxLoop
from paper_1802_03749_amd.hexloop import HexLoop
from paper_1802_03749_amd.timestep import TimeStep2D

GM1, EPS, KAPPA = 0.4, 0.25, 1.0 / 64.0
QINF = (1.0, 0.35, 0.05, 2.7)

# The benchmark's plan for AoS data; SoA data cannot use the LDS-DMA gather.
DATAFLOW = dict(schedule="dataflow", elems_per_thread=2, block_colouring="recolour")


def listed():
    return [
        # ---- edge sweeps
        # the smallest mesh of the test configurations: one launch, latency
        dict(name="edge 200x100 f64", loop="edge", nx=200, ny=100, tx=16, ty=16, order="user",
             points=2, dtype="f64", layout="aos", plan="dataflow"),
        # the block-size study's mesh, as the library partitions it
        dict(name="edge 1200x600 f64", loop="edge", nx=1200, ny=600, tx=16, ty=16,
             order="rcm+partition", points=2, dtype="f64", layout="aos", plan="dataflow"),
        # the benchmark's mesh, in the caller's own 16x16-cell blocks
        dict(name="edge 2400x1200 f64", loop="edge", nx=2400, ny=1200, tx=16, ty=16,
             order="user", points=2, dtype="f64", layout="aos", plan="dataflow"),
        # binary32 storage, odd sizes, ragged last blocks
        dict(name="edge 1133x711 f32", loop="edge", nx=1133, ny=711, tx=16, ty=16, order="user",
             points=2, dtype="f32", layout="aos", plan="dataflow"),
        # a program whose arrays are component-major
        dict(name="edge 907x613 f64 soa", loop="edge", nx=907, ny=613, tx=16, ty=16,
             order="user", points=2, dtype="f64", layout="soa", plan="dataflow"),
        # the drivers' defaults: one launch per block colour
        dict(name="edge 600x300 f64 default", loop="edge", nx=600, ny=300, tx=16, ty=16,
             order="rcm+partition", points=1, dtype="f64", layout="aos", plan="default"),
        # ---- hex sweeps
        # a large solid, with the benchmark's options
        dict(name="hex 96 f64", loop="hex", n=96, order="partition", points=3, layout="aos",
             tcmode="barrier"),
        # a small odd one that keeps its own node numbers
        dict(name="hex 33 f64 soa", loop="hex", n=33, order="partition", points=0, layout="soa",
             tcmode="lds_atomic"),
        # ---- time steps
        # a mid-size solver run with the benchmark's options
        dict(name="step 1200x600 f64 fused", loop="step", nx=1200, ny=600, order="rcm+partition",
             points=2, dtype="f64", plan="dataflow", fused=True),
        # a small odd one in binary32 storage that keeps its own point numbers
        dict(name="step 353x241 f32", loop="step", nx=353, ny=241, order="partition", points=0,
             dtype="f32", plan="dataflow", fused=False),
        # the drivers' defaults
        dict(name="step 500x400 f64 default", loop="step", nx=500, ny=400,
             order="rcm+partition", points=1, dtype="f64", plan="default", fused=False),
        # ---- a batch of small meshes of uneven size
        dict(name="batch 24 f64", loop="batch", meshes=24, c_min=2000, c_max=40000,
             size_seed=5, dtype="f64"),
    ]


def draw(rng):
    def log_uniform(a, b):
        return math.exp(rng.uniform(math.log(a), math.log(b)))

    def sides(c):
        aspect = log_uniform(0.4, 2.5)
        nx = max(40, round(math.sqrt(c * aspect)))
        return nx, max(40, round(c / nx))

    kind = rng.random()
    if kind < 0.5:
        nx, ny = sides(log_uniform(4e3, 1.1e6))
        tx, ty = rng.choice([(16, 16), (16, 16), (16, 8), (32, 16)])
        plan = rng.choice(["dataflow", "dataflow", "dataflow", "default"])
        order, points = rng.choice([("user", 2), ("user", 1), ("rcm+partition", 2),
                                    ("partition", 0)])
        return dict(loop="edge", nx=nx, ny=ny, tx=tx, ty=ty, order=order, points=points,
                    dtype=rng.choice(["f64", "f64", "f32"]),
                    layout=rng.choice(["aos", "aos", "aos", "soa"]), plan=plan)
    if kind < 0.72:
        return dict(loop="hex", n=round(log_uniform(12, 92)), order="partition",
                    points=rng.choice([0, 3, 3]), layout=rng.choice(["aos", "aos", "soa"]),
                    tcmode=rng.choice(["barrier", "lds_atomic"]))
    if kind < 0.92:
        nx, ny = sides(log_uniform(4e3, 6e5))
        return dict(loop="step", nx=nx, ny=ny,
                    **rng.choice([dict(order="rcm+partition", points=2),
                                  dict(order="partition", points=0)]),
                    dtype=rng.choice(["f64", "f32"]),
                    plan=rng.choice(["dataflow", "dataflow", "default"]),
                    fused=rng.random() < 0.6)
    return dict(loop="batch", meshes=rng.randint(4, 28), c_min=1000, c_max=30000,
                size_seed=rng.randint(1, 10 ** 6), dtype=rng.choice(["f64", "f32"]))


# ------------------------------------------------------------------ meshes
def quad(nx, ny, seed, diagonal=True):
    """A jittered nx x ny quad grid: coordinates, states, their time-step
    scalar and the maps.  The normal (y_b - y_a, x_a - x_b) of an interior
    edge points from its cell L into its cell R, that of a boundary edge out
    of the domain; a cell's nodes run counter-clockwise."""
    rng = np.random.default_rng(seed)

    def numbering(w, h):
        i, j = np.tile(np.arange(w), h), np.repeat(np.arange(h), w)
        if diagonal:
            o = np.argsort((i + j) * np.int64(h) + j, kind="stable")
            i, j = i[o], j[o]
        num = np.empty((h, w), np.int32)
        num[j, i] = np.arange(w * h, dtype=np.int32)
        return i, j, num

    ni, nj, node = numbering(nx + 1, ny + 1)
    ci, cj, cell = numbering(nx, ny)
    x = np.stack([ni, nj], 1) + np.round(rng.uniform(-0.2, 0.2, (ni.size, 2)) * 2 ** 20) / 2 ** 20
    rho, p = rng.uniform(0.9, 1.1, ci.size), rng.uniform(0.9, 1.1, ci.size)
    u, v = rng.uniform(-0.2, 0.2, ci.size), rng.uniform(-0.2, 0.2, ci.size)
    q = np.stack([rho, rho * u, rho * v, p / GM1 + 0.5 * rho * (u * u + v * v)], 1)
    # interior edges, cell by cell: the one to its right, then the one above
    sw, se, ne, nw = (node[cj, ci], node[cj, ci + 1], node[cj + 1, ci + 1], node[cj + 1, ci])
    here = np.arange(ci.size, dtype=np.int32)
    right = cell[cj, np.minimum(ci + 1, nx - 1)]
    above = cell[np.minimum(cj + 1, ny - 1), ci]
    keep = np.stack([ci + 1 < nx, cj + 1 < ny], 1).ravel()
    pick = lambda r, t: np.stack([r, t], 1).ravel()[keep]
    e2n = np.stack([pick(se, ne), pick(ne, nw)], 1)
    e2c = np.stack([pick(here, here), pick(right, above)], 1)
    # boundary edges: bottom, right, top, left
    a, b = np.arange(nx), np.arange(ny)
    b2n = np.concatenate([np.stack(s, 1) for s in (
        (node[0, a], node[0, a + 1]), (node[b, nx], node[b + 1, nx]),
        (node[ny, a + 1], node[ny, a]), (node[b + 1, 0], node[b, 0]))])
    b2c = np.concatenate([cell[0, a], cell[b, nx - 1], cell[ny - 1, a], cell[b, 0]])[:, None]
    m = SimpleNamespace(nx=nx, ny=ny, x=x, q=q, e2n=e2n, e2c=e2c, b2n=b2n, b2c=b2c,
                        c2n=np.stack([sw, se, ne, nw], 1), ci=ci, cj=cj)
    m.adt = cell_adt(m, x, q)
    return m


def hexa(n, seed):
    """A jittered n^3 hex grid, elements and nodes numbered row by row."""
    rng = np.random.default_rng(seed)
    m = n + 1
    k, j, i = np.meshgrid(*(np.arange(n, dtype=np.int32),) * 3, indexing="ij")
    base = ((k * m + j) * m + i).ravel()
    e2n = np.stack([base + o for o in (0, 1, m + 1, m, m * m, m * m + 1, m * m + m + 1,
                                       m * m + m)], 1).astype(np.int32)
    k, j, i = np.meshgrid(*(np.arange(m),) * 3, indexing="ij")
    x = np.stack([i.ravel(), j.ravel(), k.ravel()], 1) + rng.uniform(-0.1, 0.1, (m ** 3, 3))
    return SimpleNamespace(x=x, v=rng.uniform(-0.2, 0.2, (m ** 3, 3)), e2n=e2n)


def tiles(m, tx, ty):
    """The caller's blocks: an interior edge belongs to the tx x ty tile of
    cells that its cell R lies in."""
    across = -(-m.nx // tx)
    tile = (m.cj // ty) * across + m.ci // tx
    return tile[m.e2c[:, 1]].astype(np.int32)


def batch_meshes(case, seed):
    rng = np.random.default_rng(case["size_seed"])
    out = []
    for k in range(case["meshes"]):
        c = math.exp(rng.uniform(math.log(case["c_min"]), math.log(case["c_max"])))
        nx = max(2, round(math.sqrt(2.0 * c)))
        out.append(quad(nx, max(2, round(c / nx)), 1000 * seed + k))
    return out


# ------------------------------------------------------------------- passes
def prepare(case, seed):
    if case["loop"] == "edge":
        m = quad(case["nx"], case["ny"], seed)
        size = 2 * case["tx"] * case["ty"]
        kw = dict(edge_blocks=tiles(m, case["tx"], case["ty"])) if case["order"] == "user" else {}
        loop = EdgeFluxLoop(m.x, m.q, m.adt, m.e2n, m.e2c, order=case["order"], block_size=size,
                            point_reorder=case["points"], layout=case["layout"],
                            dtype=case["dtype"], **kw)
        opts = dict(DATAFLOW) if case["plan"] == "dataflow" else {}
        if opts and case["layout"] == "aos":
            opts["gather"] = "lds_dma"
        return dict(loop=loop, plan=loop.plan("hier", size, **opts), kind="edge")
    if case["loop"] == "hex":
        m = hexa(case["n"], seed)
        loop = HexLoop(m.x, m.v, m.e2n, order=case["order"], block_size=256,
                       point_reorder=case["points"], layout=case["layout"])
        plan = loop.plan("hier", 256, block_colouring="min", schedule="dataflow",
                         tcmode=case["tcmode"])
        return dict(loop=loop, plan=plan, kind="hex")
    if case["loop"] == "step":
        m = quad(case["nx"], case["ny"], seed, diagonal=case["points"] != 0)
        ts = TimeStep2D(m.x, m.q, m.e2n, m.e2c, m.b2n, m.b2c, m.c2n, QINF, order=case["order"],
                        block_size=512, point_reorder=case["points"], dtype=case["dtype"])
        opts = dict(DATAFLOW, gather="lds_dma") if case["plan"] == "dataflow" else {}
        ts.build_plans(flux_block_size=512, fuse_adt=case["fused"], **opts)
        return dict(step=ts, kind="step")
    b = BatchedSteps(batch_meshes(case, seed), QINF, mode="union", dtype=case["dtype"],
                     candidates=[dict(DATAFLOW, block_size=512, gather="lds_dma")], tune_reps=1)
    b.capture()
    return dict(batch=b, step=b.steps[0], kind="batch")


def run(state):
    kind = state["kind"]
    if kind == "edge":
        state["loop"].run(state["plan"])
        return {"res": state["loop"].res}
    if kind == "hex":
        state["loop"].run(state["plan"])
        return {"force": state["loop"].force}
    ts = state["step"]
    if kind == "step":
        ts.step()
    else:
        state["batch"].replay()
    return {"q": ts.q, "adt": ts.adt, "res": ts.res, "rms": ts.rms}


def work(case):
    """Every input read once, every output written once, the int32 maps
    included."""
    if case["loop"] == "hex":
        n = case["n"]
        return {"bytes": 96 * (n + 1) ** 3 + 32 * n ** 3, "flops": 200 * n ** 3}
    real = 8 if case["dtype"] == "f64" else 4
    if case["loop"] == "edge":
        C, N, E = measure.quad_counts(case["nx"], case["ny"])
        return {"bytes": measure.useful_bytes(N, C, E, real_bytes=real), "flops": 100 * E}
    shapes = ([(case["nx"], case["ny"])] if case["loop"] == "step" else
              [(m.nx, m.ny) for m in batch_meshes(case, 0)])
    total = {"bytes": 0, "flops": 0}
    for nx, ny in shapes:
        C, N, E = measure.quad_counts(nx, ny)
        B = 2 * (nx + ny)
        # x; q and res read and written; adt written; four maps
        total["bytes"] += (2 * real * N + (8 * real + 64 + real) * C + 16 * E + 16 * C + 12 * B)
        total["flops"] += 100 * (E + B) + 60 * C
    return total


# -------------------------------------------------------- binary64 evaluation
def cell_adt(m, x, q):
    u, v = q[:, 1] / q[:, 0], q[:, 2] / q[:, 0]
    p = GM1 * (q[:, 3] - 0.5 * (q[:, 1] * u + q[:, 2] * v))
    c = np.sqrt((1.0 + GM1) * p / q[:, 0])
    s = np.zeros(q.shape[0])
    for k in range(4):
        d = x[m.c2n[:, (k + 1) & 3]] - x[m.c2n[:, k]]
        s += np.abs(u * d[:, 1] - v * d[:, 0]) + c * np.sqrt((d ** 2).sum(1))
    return s


def flux(xa, xb, qL, qR, aL, aR):
    nx, ny = xb[:, 1] - xa[:, 1], xa[:, 0] - xb[:, 0]

    def normal_flux(q):
        u, v = q[:, 1] / q[:, 0], q[:, 2] / q[:, 0]
        p = GM1 * (q[:, 3] - 0.5 * (q[:, 1] * u + q[:, 2] * v))
        U = u * nx + v * ny
        return np.stack([q[:, 0] * U, q[:, 1] * U + p * nx, q[:, 2] * U + p * ny,
                         (q[:, 3] + p) * U], 1)

    mu = 0.5 * EPS * (aL + aR)
    return 0.5 * (normal_flux(qL) + normal_flux(qR)) + 0.5 * mu[:, None] * (qL - qR)


def added(res, at, f):
    for k in range(f.shape[1]):
        res[:, k] += np.bincount(at, f[:, k], res.shape[0])


def edge_res(m, x, q, adt):
    L, R = m.e2c[:, 0], m.e2c[:, 1]
    f = flux(x[m.e2n[:, 0]], x[m.e2n[:, 1]], q[L], q[R], adt[L], adt[R])
    res = np.zeros(q.shape)
    added(res, L, f)
    added(res, R, -f)
    return res


def caller_order(m, tx, ty, points):
    """New-to-old numbers of the cells when they are sorted, stably, by the
    blocks that access them: (number, list), or (smallest, number, list)."""
    across = -(-m.nx // tx)
    tile = lambda i, j: (j // ty) * across + i // tx
    none = np.int64(1) << 40
    i, j = m.ci.astype(np.int64), m.cj.astype(np.int64)
    lst = np.stack([np.where((i > 0) | (j > 0), tile(i, j), none),
                    np.where(i + 1 < m.nx, tile(i + 1, j), none),
                    np.where(j + 1 < m.ny, tile(i, j + 1), none)], 1)
    lst.sort(axis=1)
    lst[:, 1:][lst[:, 1:] == lst[:, :-1]] = none
    lst.sort(axis=1)
    number = (lst < none).sum(1)
    keys = [lst[:, 2], lst[:, 1], lst[:, 0], number]
    return np.lexsort(keys + [lst[:, 0]] if points == 2 else keys)


def hex_force(m):
    G = np.array([[1, 1, -1, -1, -1, -1, 1, 1], [1, -1, -1, 1, -1, 1, 1, -1],
                  [1, -1, 1, -1, 1, -1, 1, -1], [-1, 1, -1, 1, 1, -1, 1, -1]], np.float64)
    h = np.sqrt(((m.x[m.e2n[:, 6]] - m.x[m.e2n[:, 0]]) ** 2).sum(1))
    modes = np.einsum("ia,ead->eid", G, m.v[m.e2n])
    f = -KAPPA * h[:, None, None] * np.einsum("ia,eid->ead", G, modes)
    out = np.zeros(m.x.shape)
    added(out, m.e2n.ravel(), f.reshape(-1, 3))
    return out


def stored(a, dtype):
    """The values as the loop holds them."""
    return a if dtype == "f64" else a.astype(np.float32).astype(np.float64)


def one_step(m, dtype):
    x, q = stored(m.x, dtype), stored(m.q, dtype)
    adt = cell_adt(m, x, q)
    res = edge_res(m, x, q, adt)
    c = m.b2c[:, 0]
    far = np.broadcast_to(stored(np.array(QINF), dtype), (c.size, 4))
    added(res, c, flux(x[m.b2n[:, 0]], x[m.b2n[:, 1]], q[c], far, adt[c], adt[c]))
    d = res / adt[:, None]
    return x, q - d, adt, float((d * d).sum())


def exact(case, seed):
    if case["loop"] == "edge":
        if case["order"] == "rcm+partition":
            return None  # in the library's numbering of the cells
        m = quad(case["nx"], case["ny"], seed)
        res = edge_res(m, *(stored(a, case["dtype"]) for a in (m.x, m.q, m.adt)))
        if case["order"] == "user":
            res = res[caller_order(m, case["tx"], case["ty"], case["points"])]
        return {"res": torch.from_numpy(np.ascontiguousarray(
            res if case["layout"] == "aos" else res.T))}
    if case["loop"] == "hex":
        if case["points"]:
            return None  # in the library's numbering of the nodes
        f = hex_force(hexa(case["n"], seed))
        return {"force": torch.from_numpy(np.ascontiguousarray(
            f if case["layout"] == "aos" else f.T))}
    if case["loop"] == "batch":
        rms = sum(one_step(m, case["dtype"])[3] for m in batch_meshes(case, seed))
        return {"q": None, "adt": None, "res": None, "rms": torch.tensor([rms], dtype=torch.float64)}
    m = quad(case["nx"], case["ny"], seed, diagonal=case["points"] != 0)
    x, q, adt, rms = one_step(m, case["dtype"])
    out = {"q": None, "adt": None, "res": None,
           "rms": torch.tensor([rms], dtype=torch.float64)}
    if case["points"] == 0:
        # with the fused plans adt is the next step's
        out.update(q=torch.from_numpy(q), res=torch.zeros(q.shape, dtype=torch.float64),
                   adt=torch.from_numpy((cell_adt(m, x, q) if case["fused"] else adt)[:, None]))
    return out
