"""Measured workloads of the library, each one call (or one batch launch)
through the public binding `paper_1609_01490_amd.trimap`.

A case is a dict of plain values.  `listed()` names the fixed ones, `draw()`
gives further ones of the same ranges, `prepare()` builds what a program holds
before the call (inputs on the GPU, the plan, a workspace), `run()` makes one
call and returns its whole outputs, `work()` counts the bytes and operations
the task cannot do without, and `exact()` gives the floating-point results in
64 bits from plain torch.

Every case uses the lambda map, which the library is for (the other maps are
its comparison baselines), at the tiles and orders that the benchmark and the
autotuner settle on, or at the plain order of a plan made without flags.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1609_01490_amd import inputs, trimap as tm

_MODES = {"fp32": tm.EDM_FP32, "bf16x3": tm.EDM_BF16X3, "bf16": tm.EDM_BF16}

# Orders the benchmark's autotuner picks for the large sizes of each kernel.
_PAIRS = tm.FLAG_ORDER_PAIRS
_LIFE_STRIPS = (tm.FLAG_STRIP(3) | tm.FLAG_STRIP_ALIGN | tm.FLAG_LIFE_WIDE |
                tm.FLAG_XCD_SWIZZLE | tm.FLAG_ORDER_PAIRS)
_EDM_STRIPS = tm.FLAG_STRIP(4) | tm.FLAG_STRIP_COLS | tm.FLAG_XCD_SWIZZLE


def listed():
    return [
        # The smallest call: the integer body at the library's own default
        # size, where launch and dispatch latency count.
        {"name": "int32 n=2048", "kind": "xormul", "n": 2048, "ld": 2048, "tile": 16, "flags": 0},
        # A small fp32 elementwise call on plain contiguous tensors of odd
        # side: no row but the first is 16-byte aligned.
        {"name": "axpyt n=1501", "kind": "axpyt", "n": 1501, "ld": 1501, "tile": 32, "flags": 0},
        # The headline workload: 6.4 GB of traffic, bound by memory.
        {"name": "axpyt n=32768", "kind": "axpyt", "n": 32768, "ld": 32768, "tile": 128,
         "flags": _PAIRS},
        # A small cellular automaton run for many generations: a chain of
        # dependent launches, each far too small to fill the GPU.
        {"name": "life n=1000", "kind": "life", "n": 1000, "ld": 1000, "steps": 100, "tile": 64,
         "flags": tm.FLAG_LIFE_TEMPORAL, "graph": False},
        # The benchmark's automaton: many generations on a large grid.
        {"name": "life n=16384", "kind": "life", "n": 16384, "ld": 16384, "steps": 100, "tile": 64,
         "flags": _LIFE_STRIPS | tm.FLAG_LIFE_TEMPORAL, "graph": False},
        # A distance map of a few thousand points in a serving loop, with the
        # library's own scratch: four dependent launches on little data.
        {"name": "edm bf16x3 n=2000 d=64", "kind": "edm", "mode": "bf16x3", "n": 2000, "d": 64,
         "ldx": 64, "tile": 128, "flags": 0, "noalloc": True},
        # The benchmark's distance map on the matrix cores: 8.6 GB written.
        {"name": "edm bf16x3 n=65536 d=128", "kind": "edm", "mode": "bf16x3", "n": 65536, "d": 128,
         "ldx": 128, "tile": 128, "flags": _EDM_STRIPS, "noalloc": False},
        # The FP32 distance map, for users who need FP32's error on every
        # pair: bound by arithmetic.
        {"name": "edm fp32 n=16384 d=128", "kind": "edm", "mode": "fp32", "n": 16384, "d": 128,
         "ldx": 128, "tile": 128, "flags": 0, "noalloc": False},
        # Four-feature distances into a plain contiguous matrix of odd side.
        {"name": "edm4 n=10007", "kind": "edm4", "n": 10007, "ld": 10007, "tile": 64, "flags": 0},
        # Collision detection at the benchmark's size: all pairs of spheres.
        {"name": "collide n=131072", "kind": "collide", "n": 131072, "dim": 3, "tile": 128,
         "flags": 0},
        # Triangles of a neighbour graph at the benchmark's size: the
        # tetrahedral domain.
        {"name": "triangles n=8192", "kind": "triangles", "n": 8192, "tile": 64},
        # The benchmark's batch: 512 distance maps and automata of sides 64
        # to 8192 in one graph launch.
        {"name": "batch 512", "kind": "batch", "count": 512, "n_lo": 64, "n_hi": 8192, "d": 32,
         "steps": 20, "edm_tile": 64, "life_tile": 64, "flags": tm.FLAG_LIFE_TEMPORAL,
         "sizes": 160901494},
    ]


def _side(rng, lo, hi):
    """A side, log-uniform in [lo, hi]: as drawn (often odd), or rounded down
    to a multiple of 64 as sizes picked by hand often are."""
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    n = min(max(n, lo), hi)
    return n // 64 * 64 if rng.random() < 0.4 and n >= 64 else n


def _up(n, k):
    return -(-n // k) * k


def draw(rng):
    kind = rng.choice(["xormul", "axpyt", "axpyt", "life", "life", "edm", "edm", "edm", "edm4",
                       "collide", "triangles", "batch"])
    if kind == "xormul":
        n = _side(rng, 64, 8192)
        return {"kind": kind, "n": n, "ld": rng.choice([n, _up(n, 4)]),
                "tile": rng.choice([16, 32, 64]), "flags": 0}
    if kind == "axpyt":
        n = _side(rng, 64, 32768)
        tile, flags = rng.choice([(32, 0), (64, 0), (128, 0), (128, _PAIRS)])
        return {"kind": kind, "n": n, "ld": rng.choice([n, _up(n, 4)]), "tile": tile,
                "flags": flags}
    if kind == "life":
        n = _side(rng, 64, 16384)
        temporal = rng.random() < 0.75
        steps = rng.randint(1, 100 if temporal else 40)
        big = rng.random() < 0.5  # the large grids' order, or a plan's plain one
        return {"kind": kind, "n": n, "ld": rng.choice([_up(n, 4), _up(n, 16)]), "steps": steps,
                "tile": 64,
                "flags": (_LIFE_STRIPS if big else 0) | (tm.FLAG_LIFE_TEMPORAL if temporal else 0),
                "graph": (not temporal) and rng.random() < 0.5}
    if kind == "edm":
        mode = rng.choice(["fp32", "bf16x3", "bf16x3", "bf16"])
        # coordinates of space, feature vectors, embeddings; odd ones among them
        d = int(round(math.exp(rng.uniform(math.log(2), math.log(256)))))
        d = rng.choice([d, _up(d, 16)])
        hi = 16384 if mode == "fp32" else (65536 if d <= 128 else 32768)
        n = _side(rng, 64, hi)
        tile = rng.choice([64, 128]) if mode == "fp32" else 128
        flags = 0 if mode == "fp32" else rng.choice([0, _EDM_STRIPS])
        fits = mode != "fp32" and n * (_up(d, 16) * 4 + 128) < tm.EDM_NOALLOC_SCRATCH_BYTES // 2
        return {"kind": kind, "mode": mode, "n": n, "d": d, "ldx": rng.choice([d, _up(d, 4)]),
                "tile": tile, "flags": flags, "noalloc": fits and rng.random() < 0.5}
    if kind == "edm4":
        n = _side(rng, 64, 32768)
        return {"kind": kind, "n": n, "ld": rng.choice([n, _up(n, 4)]),
                "tile": rng.choice([64, 128]), "flags": 0}
    if kind == "collide":
        return {"kind": kind, "n": _side(rng, 256, 131072), "dim": rng.choice([1, 3, 3]),
                "tile": rng.choice([64, 128]), "flags": 0}
    if kind == "triangles":
        return {"kind": kind, "n": _side(rng, 128, 8192), "tile": rng.choice([32, 64, 64])}
    return {"kind": "batch", "count": int(round(math.exp(rng.uniform(math.log(8), math.log(512))))),
            "n_lo": 64, "n_hi": int(round(math.exp(rng.uniform(math.log(512), math.log(8192))))),
            "d": rng.choice([3, 16, 32]), "steps": rng.randint(4, 20), "edm_tile": 64,
            "life_tile": 64, "flags": tm.FLAG_LIFE_TEMPORAL, "sizes": rng.randrange(1 << 30)}


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _uniform(shape, g, lo, hi):
    return torch.empty(shape, dtype=torch.float32, device="cuda").uniform_(lo, hi, generator=g)


def _life_grid(n, ld, g):
    """uint8 n x ld: lower-triangle cells alive with probability 0.3."""
    grid = torch.zeros((n, ld), dtype=torch.uint8, device="cuda")
    for r0 in range(0, n, 4096):
        r1 = min(n, r0 + 4096)
        cells = (torch.rand((r1 - r0, n), device="cuda", generator=g) < 0.3).to(torch.uint8)
        grid[r0:r1, :n] = cells.tril_(r0)
    return grid


def _points(n, d, ldx, seed):
    """n x d points of row pitch ldx, uniform in [0, 1), 1 % near-duplicates."""
    X, _ = inputs.points(n, d, seed=seed)
    buf = torch.zeros((n, ldx), dtype=torch.float32, device="cuda")
    buf[:, :d] = torch.from_numpy(X).cuda()
    return buf[:, :d]


def _batch_layout(case):
    """(is_map, n, offset of its output or grid, pitch) per instance, and the
    lengths of the distance and grid arenas (every instance 256-byte aligned)."""
    rows, pairs, cells = [], 0, 0
    for kind, n in inputs.batch_instances(case["count"], case["n_lo"], case["n_hi"],
                                          seed=case["sizes"]):
        if kind == "edm":
            rows.append((True, n, pairs, case["d"]))
            pairs += _up(n * (n - 1) // 2, 64)
        else:
            rows.append((False, n, cells, _up(n, 16)))
            cells += _up(n * _up(n, 16), 256)
    return rows, pairs, cells


def _batch_points(case, rows, g):
    return [_uniform((n, case["d"]), g, 0.0, 1.0) if is_map else None
            for is_map, n, _, _ in rows]


def prepare(case, seed):
    kind = case["kind"]
    n = case.get("n")
    st = {"case": dict(case)}
    if kind == "batch":
        rows, pairs, cells = _batch_layout(case)
        g = _gen(seed)
        xs = _batch_points(case, rows, g)
        dist = torch.zeros(pairs, dtype=torch.float32, device="cuda")
        grid_a = torch.zeros(cells, dtype=torch.uint8, device="cuda")
        grid_b = torch.zeros(cells, dtype=torch.uint8, device="cuda")
        a, b = [], []
        for x, (is_map, side, at, pitch) in zip(xs, rows):
            if is_map:
                a.append(x)
                b.append(dist[at:at + side * (side - 1) // 2])
            else:
                ga = grid_a[at:at + side * pitch].view(side, pitch)
                ga.copy_(_life_grid(side, pitch, g))
                a.append(ga)
                b.append(grid_b[at:at + side * pitch].view(side, pitch))
        bt = tm.Batch([tm.KIND_EDM if r[0] else tm.KIND_LIFE for r in rows], [r[1] for r in rows],
                      [case["d"] if r[0] else 0 for r in rows], case["edm_tile"],
                      case["life_tile"], case["steps"], case["flags"])
        bt.bind(a, b)
        st.update(batch=bt, dist=dist, grids=(grid_a, grid_b))
        return st
    if kind == "triangles":
        P, r2 = inputs.points3(n, seed=seed)
        st.update(plan=tm.TetPlan(n, case["tile"], "lambda"), points=torch.from_numpy(P).cuda(),
                  r2=float(r2), counts=torch.zeros(n, dtype=torch.int32, device="cuda"),
                  total=torch.zeros(1, dtype=torch.int64, device="cuda"))
        return st
    strict = kind in ("edm", "collide")
    st["plan"] = tm.Plan(n, case["tile"], "lambda", include_diag=not strict, flags=case["flags"])
    if kind == "xormul":
        A, B, _ = inputs.int_elementwise(n, seed=seed, ld=0)
        st.update(a=torch.from_numpy(A.view(np.int32)).cuda(),
                  b=torch.from_numpy(B.view(np.int32)).cuda(),
                  c=torch.zeros((n, case["ld"]), dtype=torch.int32, device="cuda"))
    elif kind == "axpyt":
        x, y = _axpyt_inputs(case, seed)
        st.update(x=x, y=y, c=torch.zeros_like(x))
    elif kind == "life":
        cur = _life_grid(n, case["ld"], _gen(seed))
        st.update(cur=cur, nxt=torch.zeros_like(cur))
    elif kind == "edm":
        mode = _MODES[case["mode"]]
        st.update(x=_points(n, case["d"], case["ldx"], seed), mode=mode,
                  out=torch.zeros(n * (n - 1) // 2, dtype=torch.float32, device="cuda"))
        if mode != tm.EDM_FP32 and not case["noalloc"]:
            st["ws"] = torch.empty(st["plan"].edm_workspace_size(case["d"], mode),
                                   dtype=torch.uint8, device="cuda")
    elif kind == "edm4":
        st.update(p=torch.from_numpy(inputs.points4(n, seed=seed)).cuda(),
                  c=torch.zeros((n, case["ld"]), dtype=torch.float32, device="cuda"))
    else:
        st.update(s=torch.from_numpy(inputs.spheres(n, case["dim"], seed=seed)).cuda(),
                  counts=torch.zeros(n, dtype=torch.int32, device="cuda"))
    return st


def _axpyt_inputs(case, seed):
    g = _gen(seed)
    shape = (case["n"], case["ld"])
    return _uniform(shape, g, -1.0, 1.0), _uniform(shape, g, -1.0, 1.0)


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "xormul":
        st["plan"].elementwise(tm.OP_XORMUL_I32, st["a"], st["b"], st["c"])
        return st["c"]
    if kind == "axpyt":
        st["plan"].elementwise(tm.OP_AXPYT_F32, st["x"], st["y"], st["c"], a=1.25)
        return st["c"]
    if kind == "life":
        st["plan"].stencil(st["cur"], st["nxt"], case["steps"], use_graph=case["graph"])
        if case["steps"] % 2:  # the run goes on from the grid that holds the result
            st["cur"], st["nxt"] = st["nxt"], st["cur"]
        return st["cur"]
    if kind == "edm":
        if case["noalloc"]:
            st["plan"].edm_noalloc(st["x"], st["out"], st["mode"])
        else:
            st["plan"].edm(st["x"], st["out"], st["mode"], ws=st.get("ws"))
        return st["out"]
    if kind == "edm4":
        st["plan"].elementwise(tm.OP_EDM4_F32, st["p"], None, st["c"])
        return st["c"]
    if kind == "collide":
        st["plan"].collide(st["s"], st["counts"], case["dim"])
        return st["counts"]
    if kind == "triangles":
        st["plan"].triangles(st["points"], st["r2"], st["counts"], st["total"])
        return {"counts": st["counts"], "total": st["total"]}
    st["batch"].launch(tm.BATCH_GRAPH)
    return {"distances": st["dist"], "grid": st["grids"][case["steps"] % 2]}


def work(case):
    kind = case["kind"]
    n = case.get("n", 0)
    cells, pairs = n * (n + 1) // 2, n * (n - 1) // 2
    if kind == "xormul":
        return {"bytes": 4 * cells + 8 * n, "flops": 3 * cells}
    if kind == "axpyt":
        return {"bytes": 12 * cells, "flops": 2 * cells}
    if kind == "life":  # the first grid read, the last one written; 9 adds and tests a cell
        return {"bytes": 2 * cells, "flops": 9 * cells * case["steps"]}
    if kind == "edm":  # a multiply and an add per pair and dimension
        return {"bytes": 4 * pairs + 4 * n * case["d"], "flops": 2 * pairs * case["d"]}
    if kind == "edm4":
        return {"bytes": 4 * cells + 16 * n, "flops": 8 * cells}
    if kind == "collide":
        return {"bytes": 20 * n, "flops": (8 if case["dim"] == 3 else 4) * pairs}
    if kind == "triangles":  # the neighbour relation of every pair
        return {"bytes": 20 * n, "flops": 8 * pairs}
    total = {"bytes": 0, "flops": 0}
    for is_map, side, _, _ in _batch_layout(case)[0]:
        one = work({"kind": "edm" if is_map else "life", "n": side, "d": case["d"],
                    "steps": case["steps"]})
        total = {k: total[k] + one[k] for k in total}
    return total


# --------------------------------------------------------------------------
# 64-bit results
# --------------------------------------------------------------------------

def _rows(n, width):
    """Row ranges of about 2^24 cells each."""
    step = max(1, (1 << 24) // max(1, width))
    return [(r, min(n, r + step)) for r in range(0, n, step)]


def _pair_distances(a, b):
    """Distances of every row of a to every row of b, summed directly."""
    s = torch.zeros((a.shape[0], b.shape[0]), dtype=torch.float64, device=a.device)
    for k in range(a.shape[1]):
        diff = a[:, k, None] - b[None, :, k]
        s.addcmul_(diff, diff)
    return s.sqrt_()


def _condensed(x, out):
    """The strict lower triangle of the distance matrix of x, row by row."""
    x = x.double()
    n = x.shape[0]
    for r0, r1 in _rows(n, n):
        full = _pair_distances(x[r0:r1], x[:r1])
        low = torch.ones((r1 - r0, r1), dtype=torch.bool, device=x.device).tril_(r0 - 1)
        out[r0 * (r0 - 1) // 2:r1 * (r1 - 1) // 2] = full[low]
    return out


def exact(case, seed):
    """The floating-point outputs in 64 bits.  None for the integer and byte
    outputs, which are whole numbers with nothing to round."""
    kind = case["kind"]
    if kind == "axpyt":
        n, ld = case["n"], case["ld"]
        x, y = _axpyt_inputs(case, seed)
        c = torch.zeros((n, ld), dtype=torch.float64, device="cuda")
        for r0, r1 in _rows(n, n):
            c[r0:r1, :n] = (1.25 * x[r0:r1, :n].double() + y[:n, r0:r1].t().double()).tril_(r0)
        return c
    if kind == "edm4":
        n, ld = case["n"], case["ld"]
        p = torch.from_numpy(inputs.points4(n, seed=seed)).cuda().double()
        c = torch.zeros((n, ld), dtype=torch.float64, device="cuda")
        for r0, r1 in _rows(n, n):
            c[r0:r1, :n] = _pair_distances(p[r0:r1], p).tril_(r0)
        return c
    if kind == "edm":
        n = case["n"]
        out = torch.zeros(n * (n - 1) // 2, dtype=torch.float64, device="cuda")
        return _condensed(_points(n, case["d"], case["ldx"], seed), out)
    if kind == "batch":
        rows, pairs, _ = _batch_layout(case)
        out = torch.zeros(pairs, dtype=torch.float64, device="cuda")
        for x, (is_map, n, at, _) in zip(_batch_points(case, rows, _gen(seed)), rows):
            if is_map:
                _condensed(x, out[at:at + n * (n - 1) // 2])
        return {"distances": out, "grid": None}
    return None
