"""The work that programs on this framework have it do, as measurable cases.

A case is a dict of plain values: its kind (one per application or heap
service), sizes and options.  ``prepare`` builds what a program keeps (a
simulation with its heap, a captured graph, the tensors it feeds in) from a
seed; ``run`` advances it by one frame - the steps between two looks at the
state - and reads the state back through ``gather``, ordered by the objects'
ids; ``work`` says what one frame cannot do without; ``exact`` computes the
frame's floating-point outputs in float64 with plain torch.

Kinds:
  spring      SpringSim: Spring::force + Node::update steps of one or several
              spring meshes in one heap, springs breaking
  adjoint     spring_rollout, forward and backward: one optimization step over
              stiffnesses and initial velocities
  nbody       NbodySim: all-pairs force (device_do) + update steps
  gol         GolSim: births are device allocations, deaths device deletions
  generation  GenerationSim: Game of Life with dying cells, rule Burst
  wator       WatorSim: fish and sharks, created and deleted in methods
  structure   StructureSim: a pull, substeps, and the removal of disconnected
              nodes (fracture checks of a loaded, damaged structure)
  objects     Heap: parallel_new of a batch, gather of its fields, destroy
"""

import math

import numpy as np
import torch

from paper_1908_05845_amd import smmo
from paper_1908_05845_amd.adjoint import spring_rollout
from paper_1908_05845_amd.sims import GenerationSim, GolSim, NbodySim, SpringSim, StructureSim, WatorSim

DEV = "cuda"


def listed():
    return [
        # the smallest call: a mesh of a few dozen blocks stepped between two
        # frames of an interactive program; launches and latency are all of it
        {"name": "spring_33x29", "kind": "spring", "W": 33, "H": 29, "meshes": 1, "steps": 100},
        # the ordinary mesh: 1M nodes, 3M springs, the library's main workload,
        # resident in the last-level cache
        {"name": "spring_1000x1000", "kind": "spring", "W": 1000, "H": 1000, "meshes": 1, "steps": 100},
        # many uneven structures in one heap (3.5M nodes, 10M springs): the
        # throughput form, beyond the last-level cache
        {"name": "spring_batch_224", "kind": "spring", "W": 126, "H": 125, "meshes": 224, "steps": 20},
        # one training step of the differentiable mesh: 100k nodes, 200 steps,
        # checkpoints every 20
        {"name": "adjoint_316x317", "kind": "adjoint", "W": 316, "H": 317, "steps": 200, "every": 20},
        # the all-pairs force at the size where it is pure arithmetic, and a
        # small odd cluster, where the chip is not filled
        {"name": "nbody_65536", "kind": "nbody", "n": 65536, "steps": 1},
        {"name": "nbody_3001", "kind": "nbody", "n": 3001, "steps": 8},
        # Game of Life on a board that fits the caches (the three do-alls), and
        # on one whose allocator traffic is spread over the whole chip
        {"name": "gol_256x256", "kind": "gol", "W": 256, "H": 256, "gens": 25, "fused": False, "graph": False},
        {"name": "gol_4096x4096", "kind": "gol", "W": 4096, "H": 4096, "gens": 2, "fused": True, "graph": False},
        # the generational automaton replayed from a captured graph, an odd board
        {"name": "generation_511x300", "kind": "generation", "W": 511, "H": 300, "gens": 20, "graph": True},
        # predators and prey: two churning classes, eight do-alls an iteration
        {"name": "wator_1024x1024", "kind": "wator", "W": 1024, "H": 1024, "iters": 10},
        # a loaded structure of 1M nodes with missing springs: 40 substeps, then
        # the breadth-first removal of what is no longer connected
        {"name": "structure_1000x1000", "kind": "structure", "W": 1000, "H": 1000, "substeps": 40},
        # the heap as a service: a million objects created, read and destroyed
        # in an order of the program's own
        {"name": "objects_1000003", "kind": "objects", "n": 1000003},
    ]


def draw(rng):
    kind = rng.choice(["spring", "spring", "adjoint", "nbody", "gol", "gol", "generation", "wator", "structure",
                       "objects"])

    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    if kind == "spring":
        if rng.random() < 0.5:
            return {"kind": kind, "W": log_int(20, 1000), "H": log_int(20, 1000), "meshes": 1,
                    "steps": rng.randint(20, 100)}
        return {"kind": kind, "W": log_int(20, 125), "H": log_int(20, 125), "meshes": log_int(4, 200),
                "steps": rng.randint(8, 20)}
    if kind == "adjoint":
        return {"kind": kind, "W": log_int(20, 316), "H": log_int(20, 316), "steps": rng.randint(30, 200),
                "every": rng.choice([10, 20, 50])}
    if kind == "nbody":
        n = log_int(300, 65536)
        return {"kind": kind, "n": n, "steps": 1 if n > 20000 else rng.randint(1, 8)}
    if kind == "gol":
        W, H = log_int(40, 4096), log_int(40, 4096)
        return {"kind": kind, "W": W, "H": H, "gens": rng.randint(10, 25) if W * H < 1 << 20 else 2,
                "fused": rng.random() < 0.5, "graph": rng.random() < 0.5}
    if kind == "generation":
        return {"kind": kind, "W": log_int(40, 1024), "H": log_int(40, 1024), "gens": rng.randint(5, 20),
                "graph": rng.random() < 0.5}
    if kind == "wator":
        return {"kind": kind, "W": log_int(200, 1024), "H": log_int(200, 1024), "iters": rng.randint(2, 10)}
    if kind == "structure":
        return {"kind": kind, "W": log_int(40, 1000), "H": log_int(40, 1000), "substeps": rng.randint(10, 40)}
    return {"kind": kind, "n": log_int(1000, 1000000)}


# ------------------------------------------------------------------ inputs --
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _uniform(n, g, lo=0.0, hi=1.0):
    return lo + (hi - lo) * torch.rand(n, generator=g, device=DEV, dtype=torch.float64)


def _slots(ends, count):
    """For each spring end (flattened [first ends; second ends] over springs in
    id order): its rank among its node's springs by spring id."""
    S = ends[0].numel()
    node = torch.cat(ends)
    spr = torch.arange(S, device=DEV).repeat(2)
    key, order = torch.sort(node * (S + 1) + spr)
    first = torch.zeros(count + 1, dtype=torch.int64, device=DEV)
    first[1:] = torch.cumsum(torch.bincount(node, minlength=count), 0)
    rank = torch.empty_like(order)
    rank[order] = torch.arange(2 * S, device=DEV) - first[key // (S + 1)]
    return rank[:S], rank[S:]


def _spring_mesh(W, H, meshes, seed, v_sigma, weak):
    """Jittered grids with one random diagonal per cell, side by side in one
    set of arrays (device tensors).  With several meshes their heights vary
    between a quarter of H and 1.75 H, so that the batch is uneven.  A share
    `weak` of the springs starts with a strain of 0.25 to 0.35 and may break."""
    g = _gen(seed)
    if meshes == 1:
        hs = torch.tensor([H], device=DEV)
    else:                             # the sizes belong to the case, not to the seed
        spread = torch.arange(meshes, device=DEV) * 0.6180339887498949 % 1.0
        hs = (H * (0.25 + 1.5 * spread)).long().clamp(min=2)
    counts = W * hs
    N = int(counts.sum())
    off = torch.cumsum(counts, 0) - counts
    of = torch.repeat_interleave(torch.arange(meshes, device=DEV), counts)
    ids = torch.arange(N, device=DEV)
    local = ids - off[of]
    i, j, rows = local % W, local // W, hs[of]
    h = 1.0 / W
    x = ((i + 0.5 + _uniform(N, g, -0.3, 0.3)) * h - 0.5).float()
    y = ((j + 0.5 + _uniform(N, g, -0.3, 0.3)) * h - 0.5 * rows * h).float()
    has_r, has_d = i + 1 < W, j + 1 < rows
    coin = _uniform(N, g) < 0.5
    a = torch.stack([ids, ids, torch.where(coin, ids, ids + 1)], 1)
    b = torch.stack([ids + 1, ids + W, torch.where(coin, ids + W + 1, ids + W)], 1)
    ok = torch.stack([has_r, has_d, has_r & has_d], 1)
    a, b = a[ok], b[ok]
    S = a.numel()
    k = (10.0 ** _uniform(S, g, 2.0, 4.0)).float()
    L0 = torch.hypot(x[b].double() - x[a].double(), y[b].double() - y[a].double())
    L0 = torch.where(_uniform(S, g) < weak, L0 / _uniform(S, g, 1.25, 1.35), L0).float()
    sa, sb = _slots((a, b), N)
    v = v_sigma * torch.randn((2, N), generator=g, device=DEV, dtype=torch.float64)
    return {"x": x, "y": y, "vx": v[0].float(), "vy": v[1].float(), "m": torch.ones(N, device=DEV),
            "a": a.int(), "b": b.int(), "k": k, "L0": L0, "slot_a": sa.int(), "slot_b": sb.int()}


def _structure_mesh(W, H, seed):
    """Brick-wall lattice (at most three springs per node), anchored on the
    left, pulled slowly on the right, with 12 % of its springs missing and a
    few weak ones: parts of it hang loose, and a few springs fail under load."""
    g = _gen(seed)
    N = W * H
    ids = torch.arange(N, device=DEV)
    i, j = ids % W, ids // W
    h = 1.0 / W
    x = ((i + _uniform(N, g, -0.2, 0.2)) * h).float()
    y = ((j + _uniform(N, g, -0.2, 0.2)) * h).float()
    ntype = torch.full((N,), 2, dtype=torch.int32, device=DEV)
    ntype[i == W - 1] = 1
    ntype[i == 0] = 0
    hor = ids[i + 1 < W]
    ver = ids[((i + j) % 2 == 0) & (j + 1 < H)]
    p1, p2 = torch.cat([hor, ver]), torch.cat([hor + 1, ver + W])
    S = p1.numel()
    keep = _uniform(S, g) >= 0.12
    k = (10.0 ** _uniform(S, g, 2.0, 3.0)).float()
    L0 = torch.hypot(x[p2].double() - x[p1].double(), y[p2].double() - y[p1].double())
    L0 = (L0 / _uniform(S, g, 0.99, 1.01)).float()
    frail = torch.where(_uniform(S, g) < 0.001, _uniform(S, g, 0.0, 0.01), _uniform(S, g, 0.04, 0.08))
    s1, s2 = _slots((p1, p2), N)
    nspr = torch.bincount(torch.cat([p1[keep], p2[keep]]), minlength=N)
    alive = nspr > 0
    vx = torch.zeros(N, device=DEV)
    vx[ntype == 1] = 0.002
    return {"ntype": ntype, "nalive": alive.to(torch.uint8), "x": x, "y": y, "vx": vx,
            "vy": torch.zeros(N, device=DEV), "m": torch.ones(N, device=DEV), "nspr": nspr.int(),
            "p1": p1.int(), "p2": p2.int(), "k": k, "L0": L0, "maxf": (k.double() * L0.double() * frail).float(),
            "s1": s1.int(), "s2": s2.int(), "salive": keep.to(torch.uint8)}


def _host(mesh):
    return {key: v.cpu().numpy() for key, v in mesh.items()}


def _bodies(n, seed):
    g = _gen(seed)
    r, th = torch.sqrt(_uniform(n, g)), 2 * math.pi * _uniform(n, g)
    return {"x": (r * torch.cos(th)).float(), "y": (r * torch.sin(th)).float(), "vx": torch.zeros(n, device=DEV),
            "vy": torch.zeros(n, device=DEV), "m": _uniform(n, g, 0.5, 1.5).float()}


# forward steps of the library's mesh workload; a rollout that is trained on
# moves by a fraction of the spacing
SPRING = {"dt": 1e-5, "limit": 0.3, "v_sigma": 0.01, "weak": 0.005}
ROLLOUT = {"dt": 1e-4, "v_sigma": 0.05}
STRUCTURE_DT = 1e-4
NBODY_EPS, NBODY_DT = 1e-3, 1e-4
WATOR = (4, 12, 8, 4)                 # fish spawn, shark spawn, energy, boost


def _captured(step):
    """One HIP graph of what `step` launches."""
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        step(torch.cuda.current_stream())
    return g


def prepare(case, seed):
    kind = case["kind"]
    st = {"case": case}
    if kind == "spring":
        mesh = _spring_mesh(case["W"], case["H"], case["meshes"], seed, SPRING["v_sigma"], SPRING["weak"])
        st["sim"] = SpringSim(_host(mesh), SPRING["dt"], SPRING["limit"])
    elif kind == "adjoint":
        mesh = _spring_mesh(case["W"], case["H"], 1, seed, ROLLOUT["v_sigma"], 0.0)
        N = mesh["x"].numel()
        st["mesh"] = _host(mesh)
        st["k"] = mesh["k"].clone().requires_grad_()
        st["v0"] = torch.stack([mesh["vx"], mesh["vy"]], 1).requires_grad_()
        st["g"] = torch.randn((N, 2), generator=_gen(seed + 1), device=DEV)
    elif kind == "nbody":
        n = case["n"]
        st["sim"] = NbodySim(_host(_bodies(n, seed)), 1.0 / n, NBODY_EPS, NBODY_DT)
    elif kind in ("gol", "generation"):
        W, H = case["W"], case["H"]
        init = (_uniform(W * H, _gen(seed)) < 0.25).to(torch.uint8).cpu().numpy()
        if kind == "gol":
            sim = GolSim(W, H, init, fused=case["fused"])
        else:
            sim = GenerationSim(W, H, init)
        if case["graph"]:
            sim.step(2)               # every do-all has run once before the capture
            sim.heap.sync()
            st["graph"] = _captured(lambda s: sim.step(case["gens"], stream=s))
        st["sim"] = sim
    elif kind == "wator":
        W, H = case["W"], case["H"]
        g = _gen(seed)
        u, v = _uniform(W * H, g), _uniform(W * H, g)
        what = torch.where(u < 0.30, 1, torch.where(u < 0.35, 2, 0))
        limit = torch.where(what == 1, WATOR[0], WATOR[1])
        init = {"kind": what.to(torch.uint8), "timer": torch.where(what > 0, (v * (limit + 1)).long(), 0).int(),
                "energy": torch.where(what == 2, WATOR[2], 0).int()}
        st["sim"] = sim = WatorSim(W, H, seed, WATOR, _host(init))
        st["cell_of"] = torch.zeros(64 * sim.heap.blocks, dtype=torch.int64, device=DEV)
        st["cell_of"][sim.cells.long()] = torch.arange(W * H, device=DEV)
    elif kind == "structure":
        st["sim"] = StructureSim(_host(_structure_mesh(case["W"], case["H"], seed)), STRUCTURE_DT)
    else:
        n = case["n"]
        g = _gen(seed)
        fields = [("x", "f32", 1), ("y", "f32", 1), ("key", "i32", 1), ("tag", "u8", 1), ("w", "f32", 4)]
        st["heap"] = smmo.Heap({"Particle": fields}, blocks=(n + 63) // 64 + 16)
        st["values"] = {"x": torch.randn(n, generator=g, device=DEV), "y": torch.randn(n, generator=g, device=DEV),
                        "key": torch.arange(n, dtype=torch.int32, device=DEV),
                        "tag": torch.randint(0, 200, (n,), generator=g, device=DEV, dtype=torch.uint8),
                        "w": torch.randn((n, 4), generator=g, device=DEV)}
        st["order"] = torch.randperm(n, generator=g, device=DEV)
    return st


# ------------------------------------------------------------------- frames --
def _by(index, values, n):
    out = torch.zeros((n,) + values.shape[1:], dtype=values.dtype, device=values.device)
    out[index] = values
    return out


def _read(heap, cname, names, n, key="id", count=None):
    """Fields of a class's live objects ordered by their key field, zero where
    no object has the key; `count`: as many objects as there can be."""
    g = heap.gather(cname, [key] + names, capacity=n if count is None else count)
    at = g[key].long()
    return at, {f: _by(at, g[f], n) for f in names}


def _present(at, n):
    out = torch.zeros(n, dtype=torch.uint8, device=at.device)
    out[at] = 1
    return out


def run(st):
    case, kind = st["case"], st["case"]["kind"]
    if kind == "spring":
        sim = st["sim"]
        sim.step(case["steps"])
        _, out = _read(sim.heap, "Node", ["x", "y", "vx", "vy"], sim.N)
        at, forces = _read(sim.heap, "Spring", ["fx", "fy"], sim.S_all)
        return {**out, **forces, "alive": _present(at, sim.S_all)}
    if kind == "adjoint":
        st["k"].grad = st["v0"].grad = None
        xT = spring_rollout(st["k"], st["v0"], st["mesh"], ROLLOUT["dt"], case["steps"], case["every"])
        xT.backward(st["g"])
        return {"xT": xT.detach(), "gk": st["k"].grad, "gv0": st["v0"].grad}
    if kind == "nbody":
        sim = st["sim"]
        sim.step(case["steps"])
        names = ["pos_x", "pos_y", "vel_x", "vel_y", "force_x", "force_y"]
        return _read(sim.heap, "Body", names, sim.n)[1]
    if kind in ("gol", "generation"):
        sim = st["sim"]
        n = sim.W * sim.H
        if case["graph"]:
            st["graph"].replay()
        else:
            sim.step(case["gens"])
        _, out = _read(sim.heap, "Cell", ["state", "count"], n, key="cell_id")
        at, more = _read(sim.heap, "Alive", ["left"] if kind == "generation" else [], n, key="cell_id")
        return {**out, **more, "objects": _present(at, n)}
    if kind == "wator":
        sim = st["sim"]
        n = sim.W * sim.H
        sim.step(case["iters"])
        f = sim.heap.gather("Fish", ["pos", "timer"], capacity=n)
        s = sim.heap.gather("Shark", ["pos", "timer", "energy"], capacity=n)
        fc, sc = st["cell_of"][f["pos"].long()], st["cell_of"][s["pos"].long()]
        what = torch.zeros(n, dtype=torch.uint8, device=fc.device)
        what[fc] = 1
        what[sc] = 2
        timer = _by(fc, f["timer"], n)
        timer[sc] = s["timer"]
        return {"kind": what, "timer": timer, "energy": _by(sc, s["energy"], n)}
    if kind == "structure":
        sim = st["sim"]
        levels = sim.iterate(case["substeps"])
        at, out = _read(sim.heap, "Node", ["x", "y", "vx", "vy", "dist", "nspr"], sim.N)
        sat, _ = _read(sim.heap, "Spring", [], sim.S)
        return {**out, "nodes": _present(at, sim.N), "springs": _present(sat, sim.S), "levels": levels}
    heap, n = st["heap"], case["n"]
    handles = heap.new("Particle", n, **st["values"])
    _, out = _read(heap, "Particle", ["x", "y", "tag", "w"], n, key="key")
    heap.destroy("Particle", handles[st["order"]])
    return out


# --------------------------------------------------------------------- work --
def work(case):
    kind = case["kind"]
    if kind in ("spring", "adjoint"):
        N = case["W"] * case["H"] * case.get("meshes", 1)
        S, T = 3 * N, case["steps"]
        # a step: spring fields 16 B read, force 8 B written and read, endpoint
        # positions 8 B per node, node fields 20 B read and 16 B written,
        # adjacency 4 B per spring end
        step, flops = 40 * S + 44 * N, 24 * S + 12 * N
        if kind == "spring":
            return {"bytes": T * step + 2 * (20 * N + 12 * S), "flops": T * flops}
        # forward, recompute, and a reverse step (spring: 16 B fields, 8 B c
        # written and read, 8 B gk, adjacency 8 B; node: positions and w 16 B,
        # adjoints 40 B)
        return {"bytes": T * (2 * step + 40 * S + 56 * N), "flops": T * (2 * flops + 40 * S + 16 * N)}
    if kind == "nbody":
        n = case["n"]
        return {"bytes": case["steps"] * 48 * n + 2 * 28 * n, "flops": case["steps"] * 20.0 * n * n}
    if kind in ("gol", "generation"):
        n = case["W"] * case["H"]
        # a generation: per cell its id, neighbour handles and state read once,
        # its count written and read, and about a third of the cells' objects
        return {"bytes": case["gens"] * (18 * n + 12 * n // 3) + 2 * (9 + 3) * n, "flops": case["gens"] * 8.0 * n}
    if kind == "wator":
        n = case["W"] * case["H"]
        # an iteration: each cell's requests cleared, written and read twice,
        # its agent and neighbours read; half of the cells hold an agent
        return {"bytes": case["iters"] * (2 * (15 + 20) * n + 2 * 28 * n // 2) + 2 * 12 * n // 2,
                "flops": case["iters"] * 40.0 * n}
    if kind == "structure":
        N = case["W"] * case["H"]
        S = 4 * N // 3
        step = 28 * S + 8 * S + 8 * S + 44 * N
        # the search reads every node's springs and its neighbours, writes distances
        return {"bytes": case["substeps"] * step + 20 * N + 16 * S + 2 * (28 * N + 4 * S),
                "flops": case["substeps"] * (24 * S + 12 * N)}
    n = case["n"]
    return {"bytes": (2 * 29 + 2 * 29 + 4 + 8) * n, "flops": 0}


# -------------------------------------------------------------------- exact --
def _f32(v):
    return float(np.float32(v))


def _spring_force64(m, x, y, k):
    a, b = m["a"].long(), m["b"].long()
    dx, dy = x[b] - x[a], y[b] - y[a]
    ln = torch.sqrt(dx * dx + dy * dy)
    c = k * (ln - m["L0"].double()) / ln
    return a, b, ln, c * dx, c * dy


def _sum_ends(a, b, f, n):
    return torch.zeros(n, dtype=torch.float64, device=DEV).index_add_(0, a, f).index_add_(0, b, -f)


def _exact_spring(case, seed):
    m = _spring_mesh(case["W"], case["H"], case["meshes"], seed, SPRING["v_sigma"], SPRING["weak"])
    dt, limit = _f32(SPRING["dt"]), _f32(SPRING["limit"])
    x, y, vx, vy = (m[key].double() for key in ("x", "y", "vx", "vy"))
    mass, L0, N = m["m"].double(), m["L0"].double(), m["x"].numel()
    alive = torch.ones(L0.numel(), dtype=torch.bool, device=DEV)
    for _ in range(case["steps"]):
        a, b, ln, fx, fy = _spring_force64(m, x, y, m["k"].double())
        alive &= (ln - L0) / L0 <= limit
        fx, fy = torch.where(alive, fx, 0.0), torch.where(alive, fy, 0.0)
        vx = vx + _sum_ends(a, b, fx, N) / mass * dt
        vy = vy + _sum_ends(a, b, fy, N) / mass * dt
        x, y = x + vx * dt, y + vy * dt
    return {"x": x, "y": y, "vx": vx, "vy": vy, "fx": fx, "fy": fy, "alive": None}


def _exact_adjoint(case, seed):
    """The rollout in float64 and its gradients, reversed by hand step by step
    (positions of every step kept)."""
    m = _spring_mesh(case["W"], case["H"], 1, seed, ROLLOUT["v_sigma"], 0.0)
    dt, N = _f32(ROLLOUT["dt"]), m["x"].numel()
    x, y, vx, vy, k, L0, mass = (m[key].double() for key in ("x", "y", "vx", "vy", "k", "L0", "m"))
    tape = []
    for _ in range(case["steps"]):
        tape.append((x, y))
        a, b, _, fx, fy = _spring_force64(m, x, y, k)
        vx = vx + _sum_ends(a, b, fx, N) / mass * dt
        vy = vy + _sum_ends(a, b, fy, N) / mass * dt
        x, y = x + vx * dt, y + vy * dt
    g = torch.randn((N, 2), generator=_gen(seed + 1), device=DEV).double()
    lx, ly = g[:, 0].clone(), g[:, 1].clone()
    lvx, lvy, gk = torch.zeros_like(lx), torch.zeros_like(ly), torch.zeros_like(k)
    a, b = m["a"].long(), m["b"].long()
    for px, py in reversed(tape):
        lvx, lvy = lvx + dt * lx, lvy + dt * ly
        wx, wy = lvx / mass, lvy / mass
        dx, dy = px[b] - px[a], py[b] - py[a]
        ln = torch.sqrt(dx * dx + dy * dy)
        ux, uy, r = dx / ln, dy / ln, L0 / ln
        gx, gy = wx[a] - wx[b], wy[a] - wy[b]
        ug = ux * gx + uy * gy
        gk += dt * (ln - L0) * ug
        lx = lx - _sum_ends(a, b, dt * k * ((1 - r) * gx + r * ux * ug), N)
        ly = ly - _sum_ends(a, b, dt * k * ((1 - r) * gy + r * uy * ug), N)
    return {"xT": torch.stack([x, y], 1), "gk": gk, "gv0": torch.stack([lvx, lvy], 1)}


def _exact_nbody(case, seed):
    n = case["n"]
    s = {key: v.double() for key, v in _bodies(n, seed).items()}
    x, y, vx, vy, m = (s[key] for key in ("x", "y", "vx", "vy", "m"))
    G, eps2, dt = _f32(1.0 / n), _f32(NBODY_EPS) ** 2, _f32(NBODY_DT)
    for _ in range(case["steps"]):
        fx, fy = torch.empty_like(x), torch.empty_like(y)
        for lo in range(0, n, 2048):
            dx, dy = x[None] - x[lo:lo + 2048, None], y[None] - y[lo:lo + 2048, None]
            w = (dx * dx + dy * dy + eps2) ** -1.5 * m[None]
            fx[lo:lo + 2048], fy[lo:lo + 2048] = (dx * w).sum(1), (dy * w).sum(1)
        fx, fy = G * m * fx, G * m * fy
        vx, vy = vx + fx / m * dt, vy + fy / m * dt
        x, y = x + vx * dt, y + vy * dt
    return {"pos_x": x, "pos_y": y, "vel_x": vx, "vel_y": vy, "force_x": fx, "force_y": fy}


def _exact_structure(case, seed):
    m = _structure_mesh(case["W"], case["H"], seed)
    dt, N = _f32(STRUCTURE_DT), m["x"].numel()
    a, b = m["p1"].long(), m["p2"].long()
    x, y, vx, vy, mass, k, L0, maxf = (m[key].double() for key in ("x", "y", "vx", "vy", "m", "k", "L0", "maxf"))
    free, nodes = m["ntype"] == 2, m["nalive"].bool()
    pull = m["ntype"] == 1
    live = m["salive"].bool()
    x = torch.where(pull, x + vx * _f32(STRUCTURE_DT * case["substeps"]), x)
    for _ in range(case["substeps"]):
        dx, dy = x[b] - x[a], y[b] - y[a]
        ln = torch.sqrt(dx * dx + dy * dy)
        f = k * (ln - L0)
        live &= ~((ln > L0) & (f > maxf))
        c = torch.where(live & (ln > L0), f / ln, 0.0)
        vx = torch.where(free, vx + _sum_ends(a, b, c * dx, N) / mass * dt, vx)
        vy = torch.where(free, vy + _sum_ends(a, b, c * dy, N) / mass * dt, vy)
        x, y = torch.where(free, x + vx * dt, x), torch.where(free, y + vy * dt, y)
    # what the anchors reach over the live springs
    seen = (m["ntype"] == 0) & nodes
    la, lb = a[live], b[live]
    while True:
        before = int(seen.sum())
        for _ in range(16):
            hit = seen[la] | seen[lb]
            seen[la[hit]] = True
            seen[lb[hit]] = True
        if int(seen.sum()) == before:
            break
    out = {"x": x, "y": y, "vx": vx, "vy": vy}
    return {**{key: torch.where(seen & free, v, 0.0) for key, v in out.items()},
            "dist": None, "nspr": None, "nodes": None, "springs": None, "levels": None}


def exact(case, seed):
    kind = case["kind"]
    if kind == "spring":
        return _exact_spring(case, seed)
    if kind == "adjoint":
        return _exact_adjoint(case, seed)
    if kind == "nbody":
        return _exact_nbody(case, seed)
    if kind == "structure":
        return _exact_structure(case, seed)
    if kind == "objects":
        v = prepare(case, seed)["values"]
        return {"x": v["x"].double(), "y": v["y"].double(), "tag": None, "w": v["w"].double()}
    return None                       # whole numbers only
