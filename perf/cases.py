"""The workloads whose speed this repository looks after, as a user's program
runs them: calls of the tensor interface on inputs that are already on the
GPU.

listed() names them, draw() gives more of the same ranges, prepare() makes
what a program holds before the call, run() is one pass, exact() says what the
floating-point outputs are and work() what a pass cannot do without.  Inputs
follow the generators of `synth`, drawn on the GPU.
"""
import math

import numpy as np
import torch

import paper_2110_00511_amd as ash

DEVICE = "cuda"
DTYPES = {"f32": torch.float32, "f16": torch.float16, "u8": torch.uint8, "i64": torch.int64}


def listed():
    return [
        # The smallest batches (Setup 1 at c = 10^3): every call of the map's
        # life, where latency and launches are all there is.
        dict(name="cycle_1k", kind="cycle", n=1000, rho=0.99, key_dim=3, dtype="f32", elems=1, width=4, group=4,
             load=0.5, gather=True, again=True),
        # One frame's worth of keys on the default table (the 65,536-key
        # sequence of the parity tests): insert, find with values, erase, and
        # an insert that takes the erased slots again.
        dict(name="cycle_65k", kind="cycle", n=65536, rho=0.88, key_dim=3, dtype="f32", elems=1, width=4, group=4,
             load=0.5, gather=True, again=True),
        # A hash set of scalar keys at Setup 2's largest capacity, an odd count.
        dict(name="set_1m", kind="cycle", n=1000003, rho=0.5, key_dim=1, dtype="f32", elems=0, width=4, group=4,
             load=0.5, gather=False, again=False),
        # The benchmark's step: 10M keys, half of them repeats, 32-byte rows,
        # 10M finds, 5M erases, on the table shape its tuner picks.
        dict(name="cycle_10m", kind="cycle", n=10000000, rho=0.5, key_dim=3, dtype="f32", elems=8, width=2, group=1,
             load=0.85, gather=False, again=False),
        # Bulk construction: nearly all keys new, a scalar value each, default
        # table.
        dict(name="build_10m", kind="build", n=10000000, rho=0.99, key_dim=3, dtype="f32", elems=1, width=4, group=4,
             load=0.5),
        # Voxel blocks of 8^3 floats (Listing 2): rows of 2 KB stored and read
        # back.
        dict(name="blocks_2kb", kind="build_find", n=200000, rho=0.99, key_dim=3, dtype="f32", elems=512, width=4,
             group=4, load=0.5),
        # One 640 x 480 depth frame at 1 cm, points in scan order.
        dict(name="voxel_frame", kind="voxel", n=307200, voxel=0.01, order="scan"),
        # A whole scan, fine voxels (almost every point its own) and coarse
        # ones (27 points each).
        dict(name="voxel_5mm", kind="voxel", n=5000000, voxel=0.005, order="surface"),
        dict(name="voxel_5cm", kind="voxel", n=5000000, voxel=0.05, order="surface"),
        # Radius-1 neighborhoods of every surface cell (Listing 3).
        dict(name="neighbors_27", kind="neighbors", n=1250000, hood="radius", radius=1, key_dim=3, width=4, group=1,
             load=0.5),
        # 64 maps of uneven sizes in one call.
        dict(name="batched_64", kind="batched", maps=64, lo=1000, hi=1000000, elems=8, width=2, group=1, load=0.5),
        # A burst of requests of uneven sizes on a served map.
        dict(name="served_burst", kind="served", requests=400, lo=256, hi=262144, preload=4000000, elems=8, width=4,
             group=1, load=0.5),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    shapes = [(4, 4, 0.5), (2, 1, 0.85), (4, 1, 0.5), (8, 1, 0.7), (8, 8, 0.5), (16, 16, 0.7)]
    kind = rng.choice(["cycle", "cycle", "cycle", "build", "build_find", "voxel", "voxel", "neighbors", "batched",
                       "served"])
    w, g, load = rng.choice(shapes)
    shape = dict(width=w, group=g, load=load)
    if kind == "cycle":
        dtype, elems = rng.choice([("f32", 0), ("f32", 1), ("f32", 8), ("f32", 32), ("f32", 3), ("f16", 4), ("u8", 3),
                                   ("i64", 2)])
        n = _log(rng, 300, 10000000 if elems <= 8 else 2000000)
        gather = elems > 0 and n <= 2000000 and rng.random() < 0.5
        return dict(kind=kind, n=n, rho=rng.choice([0.1, 0.3, 0.5, 0.9, 0.99]), key_dim=rng.choice([1, 2, 3, 3, 3, 4]),
                    dtype=dtype, elems=elems, gather=gather, again=n <= 2000000 and rng.random() < 0.5, **shape)
    if kind == "build":
        return dict(kind=kind, n=_log(rng, 1000, 10000000), rho=rng.choice([0.5, 0.9, 0.99]),
                    key_dim=rng.choice([1, 2, 3, 3, 4]), dtype="f32", elems=rng.choice([0, 1, 4, 8]), **shape)
    if kind == "build_find":
        elems = rng.choice([48, 64, 100, 256, 512, 1024, 1536, 4096])
        return dict(kind=kind, n=_log(rng, 1000, 102400000 // elems), rho=rng.choice([0.3, 0.99]), key_dim=3, dtype="f32",
                    elems=elems, **shape)
    if kind == "voxel":
        return dict(kind=kind, n=_log(rng, 2000, 5000000), voxel=round(math.exp(rng.uniform(math.log(0.005),
                    math.log(0.2))), 4), order=rng.choice(["scan", "surface", "shuffled"]))
    if kind == "neighbors":
        hood, radius = rng.choice([("radius", 1), ("ring", 1), ("cube", 1), ("radius", 2)])
        w, g, load = rng.choice(shapes[:4])
        return dict(kind=kind, n=_log(rng, 1000, 1250000 if radius == 1 else 250000), hood=hood, radius=radius,
                    key_dim=3, width=w, group=g, load=load)
    w, g, load = rng.choice(shapes[:4])
    if kind == "batched":
        return dict(kind=kind, maps=rng.randint(2, 64), lo=_log(rng, 100, 1000), hi=_log(rng, 10000, 1000000),
                    elems=rng.choice([1, 8]), width=w, group=g, load=load)
    return dict(kind=kind, requests=rng.randint(20, 400), lo=256, hi=_log(rng, 4096, 262144),
                preload=_log(rng, 100000, 4000000), elems=rng.choice([1, 8]), width=w, group=g, load=load)


# -- inputs ------------------------------------------------------------------


def _gen(seed, salt=0):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(int(seed) * 1000003 + salt)
    return g


def _cells_for(n, rho):
    """Cells of which n uniform draws hit about rho * n distinct ones."""
    lo, hi = 1e-9, 1e3
    for _ in range(200):
        x = 0.5 * (lo + hi)
        if (1.0 - math.exp(-x)) / x > rho:
            lo = x
        else:
            hi = x
    return n / (0.5 * (lo + hi))


def _side(n, rho, dims):
    return max(2, int(round(_cells_for(n, rho) ** (1.0 / dims))))


def _keys(g, n, dims, side, lo=0):
    return torch.randint(lo, lo + side, (n, dims), dtype=torch.int32, device=DEVICE, generator=g)


def _half_hits(g, keys, n, dims, side):
    """n keys, half of them drawn from `keys`, half from a cube beside it."""
    half = n // 2
    hit = keys[torch.randint(0, keys.shape[0], (half,), device=DEVICE, generator=g)]
    q = torch.cat([hit, _keys(g, n - half, dims, side, side)])
    return q[torch.randperm(n, device=DEVICE, generator=g)].contiguous()


def _rows(g, n, case):
    dt, e = DTYPES[case["dtype"]], case["elems"]
    if not e:
        return []
    if dt.is_floating_point:
        return [torch.randn((n, e), dtype=torch.float32, device=DEVICE, generator=g).to(dt)]
    return [torch.randint(0, 256, (n, e), dtype=dt, device=DEVICE, generator=g)]


def _map(case, capacity):
    specs = [(DTYPES[case.get("dtype", "f32")], case["elems"])] if case.get("elems") else []
    m = ash.HashMap(capacity, case.get("key_dim", 3), specs, bucket_width=case["width"], probe_group=case["group"],
                    max_load=case["load"])
    m.key_buffer().zero_()  # rows that no key has taken yet are part of what a pass returns
    for j in range(len(specs)):
        m.value_buffer(j).zero_()
    return m


def _state_views(m):
    return dict(heap=m.heap_buffer(), keys=m.key_buffer(), values=[m.value_buffer(j) for j in range(len(m.value_specs))])


def _points(seed, n, order):
    """Points on spheres and rectangles in a 10 m box with 1 cm of noise, the
    surfaces one after another (random within a surface), in the order of a
    raster over each surface, or shuffled.  The set of points follows from n
    alone (so the number of voxels does too); the seed sets their order and
    which axis is which."""
    rng = np.random.default_rng(n)
    g = _gen(n, 1)
    own = np.random.default_rng(seed)
    shapes = []
    for _ in range(20):
        if rng.random() < 0.5:
            r = rng.uniform(0.3, 2.0)
            shapes.append(("sphere", rng.uniform(r, 10.0 - r, size=3), r, 4.0 * math.pi * r * r))
        else:
            a, b = rng.uniform(1.0, 4.0, size=2)
            nrm = rng.standard_normal(3)
            nrm /= np.linalg.norm(nrm)
            u = np.cross(nrm, [1.0, 0.0, 0.0] if abs(nrm[0]) < 0.9 else [0.0, 1.0, 0.0])
            u /= np.linalg.norm(u)
            shapes.append(("plane", rng.uniform(2.0, 8.0, size=3), (a, b, u, np.cross(nrm, u)), a * b))
    areas = np.array([s[3] for s in shapes])
    counts = np.floor(n * areas / areas.sum()).astype(np.int64)
    counts[np.argmax(counts)] += n - counts.sum()
    out = []
    for (kind, c, prm, _), k in zip(shapes, counts):
        k = int(k)
        if k == 0:
            continue
        if order == "scan":
            cols = max(1, int(math.sqrt(k)))
            at = torch.arange(k, device=DEVICE)
            s, t = (at // cols).double() / max(1, -(-k // cols)), (at % cols).double() / cols
        else:
            s, t = torch.rand((2, k), dtype=torch.float64, device=DEVICE, generator=g)
        if kind == "sphere":
            z, phi = 2.0 * s - 1.0, 2.0 * math.pi * t
            rad = torch.sqrt((1.0 - z * z).clamp_min(0.0))
            p = prm * torch.stack([rad * torch.cos(phi), rad * torch.sin(phi), z], 1)
        else:
            a, b, u, v = prm
            p = ((s - 0.5) * a)[:, None] * torch.from_numpy(u).to(DEVICE) + \
                ((t - 0.5) * b)[:, None] * torch.from_numpy(v).to(DEVICE)
        p = p + torch.from_numpy(c).to(DEVICE)
        out.append(p + 0.01 * torch.randn((k, 3), dtype=torch.float64, device=DEVICE, generator=g))
    if order == "scan":  # each surface's raster starts somewhere else
        out = [torch.roll(p, int(own.integers(p.shape[0])), 0) for p in out]
    else:
        out = [p[torch.randperm(p.shape[0], device=DEVICE, generator=_gen(seed, 3 + i))] for i, p in enumerate(out)]
    pts = torch.cat([out[i] for i in own.permutation(len(out))]).float()
    if order == "shuffled":
        pts = pts[torch.randperm(n, device=DEVICE, generator=_gen(seed, 2))]
    return pts[:, own.permutation(3).tolist()].contiguous()


def _cycle_inputs(case, seed):
    n, d = case["n"], case["key_dim"]
    g = _gen(seed)
    side = _side(n, case["rho"], d)
    s = dict(keys=_keys(g, n, d, side), side=side)
    s["rows"] = _rows(g, n, case)
    if case["kind"] != "build":
        s["find"] = _half_hits(g, s["keys"], n, d, side)
    if case["kind"] == "cycle":
        s["erase"] = s["keys"][torch.randperm(n, device=DEVICE, generator=g)[: n // 2]].contiguous()
        if case["again"]:
            s["more"] = _half_hits(g, s["erase"], n, d, side)
            s["more_rows"] = _rows(g, n, case)
    return s


def _served_inputs(case, seed):
    rng = np.random.default_rng(case["requests"])  # kinds and sizes follow from the case, keys from the seed
    g = _gen(seed)
    cells = max(2 * case["preload"], 64)
    side = int(math.ceil(cells ** (1.0 / 3.0)))
    code = torch.randperm(side ** 3, device=DEVICE, generator=g)[: case["preload"]]
    pre = torch.stack([code // (side * side), code // side % side, code % side], 1).int().contiguous()
    kinds = rng.choice(3, size=case["requests"], p=[0.6, 0.3, 0.1])  # find, insert, erase
    sizes = np.exp(rng.uniform(math.log(case["lo"]), math.log(case["hi"]), size=case["requests"])).astype(np.int64)
    reqs = []
    for kind, n in zip(kinds, sizes):
        r = dict(kind=int(kind), keys=_keys(g, int(n), 3, side))
        if kind == 1:
            r["rows"] = [torch.randn((int(n), case["elems"]), device=DEVICE, generator=g)]
        reqs.append(r)
    return pre, side, reqs


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("cycle", "build", "build_find"):
        s = _cycle_inputs(case, seed)
        m = _map(case, _capacity(case))
        s.update(case=case, map=m, state=_state_views(m))
        return s
    if kind == "voxel":
        return dict(case=case, points=_points(seed, case["n"], case["order"]))
    if kind == "neighbors":
        cell = 0.005
        pts = _points(seed, int(1.05 * case["n"]) + 64, "surface").double()
        cells = torch.round(pts / cell).int()
        code = (cells.long() * torch.tensor([1 << 40, 1 << 20, 1], device=DEVICE)).sum(1)
        _, inv = torch.unique(code, return_inverse=True)
        first = torch.full((int(inv.max()) + 1,), cells.shape[0], device=DEVICE).scatter_reduce(
            0, inv, torch.arange(cells.shape[0], device=DEVICE), "amin")
        cells = cells[torch.sort(first).values][: case["n"]].contiguous()
        m = ash.HashSet(2 * case["n"], 3, bucket_width=case["width"], probe_group=case["group"], max_load=case["load"])
        m.activate(cells)
        return dict(case=case, map=m, cells=cells, offsets=ash.neighbor_offsets(case["hood"], case["radius"]))
    if kind == "batched":
        rng = np.random.default_rng(case["maps"])  # the sizes follow from the case, keys from the seed
        g = _gen(seed)
        ops = []
        for _ in range(case["maps"]):
            u = int(round(math.exp(rng.uniform(math.log(case["lo"]), math.log(case["hi"])))))
            side = _side(2 * u, 0.5, 3)
            keys = _keys(g, 2 * u, 3, side)
            ops.append(dict(map=_map(case, 2 * u), insert_keys=keys,
                            insert_values=[torch.randn((2 * u, case["elems"]), device=DEVICE, generator=g)],
                            find_keys=_half_hits(g, keys, 2 * u, 3, side)))
        return dict(case=case, ops=ops)
    pre, side, reqs = _served_inputs(case, seed)
    # room for every cell the requests can name and every position of a burst's inserts
    m = _map(case, side ** 3 + sum(r["keys"].shape[0] for r in reqs if r["kind"] == 1))
    m.insert(pre, [torch.randn((pre.shape[0], case["elems"]), device=DEVICE, generator=_gen(seed, 2))])
    torch.cuda.synchronize()
    srv = ash.Server(m)
    calls, keep, outs = [], [], []
    total = sum(r["keys"].shape[0] for r in reqs)
    idx = torch.full((total,), -1, dtype=torch.int32, device=DEVICE)
    mask = torch.zeros(total, dtype=torch.uint8, device=DEVICE)
    at = 0
    for r in reqs:
        n = r["keys"].shape[0]
        o = idx[at: at + n] if r["kind"] != 2 else None
        c, k = srv.request(r["kind"], r["keys"], r.get("rows", ()), o, mask[at: at + n])
        calls.append(c)
        keep.append((r, k))
        at += n
    return dict(case=case, server=srv, map=m, calls=calls, keep=keep, idx=idx, mask=mask,
                arrivals=np.zeros(len(calls)), state=_state_views(m))


def _capacity(case):
    # twice the nominal distinct count; room for the second insert's new keys
    c = int(2 * round(case["rho"] * case["n"])) if case["rho"] <= 0.5 else int(1.2 * case["n"])
    return max(c, 64) + (case["n"] if case.get("again") else 0)


# -- one pass ----------------------------------------------------------------


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind in ("cycle", "build", "build_find"):
        m = state["map"]
        m.clear()
        out = {}
        if state["rows"]:
            out["insert"] = list(m.insert(state["keys"], state["rows"]))
        else:
            out["insert"] = list(m.activate(state["keys"]))
        if kind != "build":
            out["find"] = list(m.find(state["find"], gather=kind == "build_find" or case["gather"]))
        if kind == "cycle":
            out["erase"] = m.erase(state["erase"])
            if case["again"]:
                if state["rows"]:
                    out["more"] = list(m.insert(state["more"], state["more_rows"]))
                else:
                    out["more"] = list(m.activate(state["more"]))
        out["state"] = state["state"]
        return out
    if kind == "voxel":
        return list(ash.voxelize(state["points"], case["voxel"]))
    if kind == "neighbors":
        return list(state["map"].find_offsets(state["cells"], state["offsets"]))
    if kind == "batched":
        for op in state["ops"]:
            op["map"].clear()
        got = ash.batched(state["ops"])
        return dict(insert_idx=_one([r["insert_idx"] for r in got]), insert_mask=_one([r["insert_mask"] for r in got]),
                    find_idx=_one([r["find_idx"] for r in got]), find_mask=_one([r["find_mask"] for r in got]))
    state["server"].replay(state["calls"], state["arrivals"])
    return dict(idx=state["idx"], mask=state["mask"], state=state["state"])


def _one(parts):
    """The maps' results one after another, as a program that goes on with all maps at once takes them."""
    return torch.cat(parts)


# -- what the floating-point outputs are ---------------------------------------


def _firsts(keys):
    """(positions of the first occurrences in order, unique id per position
    ranked by first occurrence) of int32 key rows."""
    k = keys.long()
    code = k[:, 0]
    for d in range(1, k.shape[1]):
        lo = k[:, d] - k[:, d].min()
        _, code = torch.unique(code, return_inverse=True)
        code = code * (lo.max() + 1) + lo
    _, inv = torch.unique(code, return_inverse=True)
    first = torch.full((int(inv.max()) + 1,), keys.shape[0], device=keys.device).scatter_reduce(
        0, inv, torch.arange(keys.shape[0], device=keys.device), "amin")
    order = torch.argsort(first)
    rank = torch.empty_like(order)
    rank[order] = torch.arange(order.numel(), device=keys.device)
    return first[order], rank[inv]


def exact(case, seed):
    """The value rows a pass stores and gathers (plain torch); nothing for the
    other outputs, which are whole numbers."""
    if case["kind"] not in ("build", "build_find", "cycle") or not case["elems"] or case["dtype"] not in ("f32", "f16"):
        return None
    if case.get("again"):
        return None if not case["gather"] else _exact_find(case, _cycle_inputs(case, seed), stored=False)
    return _exact_find(case, _cycle_inputs(case, seed), stored=True)


def _exact_find(case, s, stored):
    n, c = case["n"], _capacity(case)
    rows = s["rows"][0].double()
    first, _ = _firsts(s["keys"])
    out = dict(insert=[None, None], state=dict(heap=None, keys=None, values=[None]))
    if stored:
        vb = torch.zeros((c, case["elems"]), dtype=torch.float64, device=DEVICE)
        vb[: first.numel()] = rows[first]
        out["state"]["values"] = [vb]
    if case["kind"] == "cycle":
        out["erase"] = None
    if case.get("again"):
        out["more"] = [None, None]
    if case["kind"] != "build":
        out["find"] = [None, None]
        if case["kind"] == "build_find" or case["gather"]:
            first, rank = _firsts(torch.cat([s["keys"], s["find"]]))
            src = first[rank[n:]]  # where each find key first occurs in keys ++ finds
            got = torch.zeros((n, case["elems"]), dtype=torch.float64, device=DEVICE)
            hit = src < n
            got[hit] = rows[src[hit]]
            out["find"] = [None, None, [got]]
    return out


# -- what a pass cannot do without -----------------------------------------------


def work(case):
    """Bytes: inputs read once, outputs and stored state written once."""
    kind = case["kind"]
    if kind in ("cycle", "build", "build_find"):
        n, u = case["n"], case["rho"] * case["n"]
        key = 4 * case["key_dim"]
        row = case["elems"] * torch.empty(0, dtype=DTYPES[case["dtype"]]).element_size()
        slot = key + 4
        b = n * (key + 5) + u * (slot + key + 4 + 2 * row)  # insert: keys, idx, mask; new slots, keys, heap, rows
        if kind != "build":
            b += n * (key + 5) + n * slot
            if kind == "build_find" or case["gather"]:
                b += n // 2 * 2 * row
        if kind == "cycle":
            b += n // 2 * (key + 1) + n // 2 * slot
            if case["again"]:
                b += n * (key + 5) + 0.8 * n * (slot + key + 4 + 2 * row)
        return dict(bytes=float(b), flops=0.0)
    if kind == "voxel":
        # points in, a voxel id each out; a key and a count per voxel (at most one per point)
        return dict(bytes=float(case["n"] * (12 + 4)), flops=0.0)
    if kind == "neighbors":
        k = {"radius": (2 * case["radius"] + 1) ** 3, "ring": 6, "cube": 8}[case["hood"]]
        return dict(bytes=float(case["n"] * (12 + 16) + case["n"] * k * 5), flops=0.0)
    if kind == "batched":
        n = case["maps"] * 2.0 * (case["hi"] - case["lo"]) / math.log(case["hi"] / case["lo"])  # mean of a log-uniform
        return dict(bytes=n * (17 + 0.5 * (16 + 16 + 8 * case["elems"]) + 17 + 16), flops=0.0)
    n = case["requests"] * (case["hi"] - case["lo"]) / math.log(case["hi"] / case["lo"])
    return dict(bytes=n * (17 + 16), flops=0.0)
