"""Performance cases: the work a user of the canvas engine has it do, through
the calls of ``paper_2203_14362_amd.spade``; where the number of results
depends on the data, through the same library's C calls (``include/spade.h``)
into output arrays that the program keeps, as a C program makes them.

Sizes and data laws are those of the repository's own configurations
(``workloads/configs.py``) and of ``bench.py``'s legs, scaled to inputs that
are quick to make: taxi-like points (a mixture of 32 anisotropic Gaussians
over a 60 x 60 km extent), tessellations whose neighbours share jittered
edges, star-shaped selection polygons with 30 % radius noise, road-like
polylines and disks around places.  Inputs are made on the GPU from the
seed alone; polygons are resident (``Context.polys``), as in the bench.

Every output is whole numbers (counts and ids), decided exactly by the
library, so ``exact`` has nothing to give: they are compared as they are.
"""
import ctypes
import math

import numpy as np
import torch

from paper_2203_14362_amd import spade

EXTENT = 60000.0   # metres
COMPONENTS = 32


def listed():
    return [
        # The smallest call: 100k uniform points against 64 zones, one plain
        # call; launches and latency count.
        {"name": "count_small", "kind": "count", "points": 100_000, "grid": 8, "vmin": 8, "vmax": 64,
         "law": "uniform", "ppv": 256.0},
        # The headline: 100M taxi-like points counted per neighbourhood,
        # polygons rasterised in the call.
        {"name": "count_zones", "kind": "count", "points": 100_000_000, "grid": 16, "vmin": 50, "vmax": 500,
         "law": "zones", "ppv": 96.0},
        # Counting per census block: more polygons than the LDS histogram
        # holds, cells small where the points are; an odd number of points.
        {"name": "count_census", "kind": "count", "points": 30_000_001, "grid": 200, "vmin": 4, "vmax": 40,
         "law": "census", "ppv": 96.0},
        # Which neighbourhood each point lies in: all (point, polygon) pairs.
        {"name": "pairs_zones", "kind": "pairs", "points": 50_000_000, "grid": 16, "vmin": 50, "vmax": 500,
         "law": "zones", "ppv": 96.0},
        # One large selection with a ragged 10k-vertex polygon.
        {"name": "select_star", "kind": "select", "points": 200_000_000, "vertices": 10_000, "area": 0.15,
         "ppv": 1600.0},
        # A served selection: one request over the resident table, its
        # polygon rasterised into the worker's canvas set.
        {"name": "serve_select", "kind": "batch_select", "points": 50_000_000, "queries": 1, "vmin": 400,
         "vmax": 400, "amin": 4e-3, "amax": 4e-3, "ppv": 96.0},
        # A batch of selections of all sizes over the resident table.
        {"name": "batch_select", "kind": "batch_select", "points": 50_000_000, "queries": 128, "vmin": 8,
         "vmax": 20_000, "amin": 1e-4, "amax": 0.15, "ppv": 24.0},
        # A served join-count: the request's tessellation is cached as a
        # canvas set and counted over the resident table.
        {"name": "serve_count", "kind": "batch_count", "points": 50_000_000, "grid": 50, "vmin": 4, "vmax": 40,
         "law": "census", "ppv": 96.0},
        # Join pairs of heavily overlapping polygons through the layer index.
        {"name": "layered_pairs", "kind": "layered", "points": 20_000_000, "polygons": 260, "vmin": 50, "vmax": 500,
         "amin": 1e-3, "amax": 2e-2, "ppv": 96.0},
        # All points within 300 m of 10,000 places.
        {"name": "disk_join", "kind": "disk_join", "points": 30_000_000, "disks": 10_000, "radius": 300.0},
        # The points within 50 m of 200 roads.
        {"name": "near_lines", "kind": "near_lines", "points": 50_000_000, "lines": 200, "vertices": 120,
         "radius": 50.0, "ppv": 96.0},
        # The 1,000 points nearest to a place.
        {"name": "knn", "kind": "knn", "points": 100_000_000, "k": 1000},
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["count", "count", "pairs", "select", "batch_select", "batch_select", "batch_count", "layered",
                       "disk_join", "near_lines", "knn"])
    c = {"kind": kind, "points": log_int(60_000, 50_000_000) | 1}
    if kind in ("count", "pairs", "batch_count"):
        law = rng.choice(["zones", "census"]) if kind != "pairs" else "zones"
        c["law"] = law
        c["grid"] = log_int(5, 30) if law == "zones" else log_int(8, 200)
        c["vmin"], c["vmax"] = (50, rng.randrange(100, 501)) if law == "zones" else (4, rng.randrange(16, 41))
        c["ppv"] = 96.0
    elif kind == "select":
        c["vertices"] = log_int(8, 20_000)
        c["area"] = math.exp(rng.uniform(math.log(1e-3), math.log(0.15)))
        c["ppv"] = rng.choice([96.0, 384.0, 1600.0])
    elif kind == "batch_select":
        c["queries"] = log_int(1, 96)
        c["vmin"], c["vmax"], c["amin"], c["amax"] = 8, 20_000, 1e-4, 0.15
        c["ppv"] = rng.choice([24.0, 96.0])
    elif kind == "layered":
        c["points"] = log_int(60_000, 15_000_000) | 1
        c["polygons"] = log_int(20, 260)
        c["vmin"], c["vmax"], c["amin"], c["amax"] = 50, 500, 1e-3, 2e-2
        c["ppv"] = 96.0
    elif kind == "disk_join":
        c["points"] = log_int(60_000, 20_000_000) | 1
        c["disks"] = log_int(10, 10_000)
        c["radius"] = float(rng.randrange(50, 301))
    elif kind == "near_lines":
        c["lines"] = log_int(1, 300)
        c["vertices"] = log_int(2, 200)
        c["radius"] = float(rng.randrange(5, 101))
        c["ppv"] = 96.0
    else:
        c["k"] = log_int(1, 5000)
    return c


# ---------------------------------------------------------------- inputs

def _mixture(rng):
    """The taxi-like mixture's parameters."""
    return {"w": rng.dirichlet(np.ones(COMPONENTS)), "c": rng.uniform(0.1 * EXTENT, 0.9 * EXTENT, (COMPONENTS, 2)),
            "s": rng.uniform(200.0, 3000.0, (COMPONENTS, 2)), "th": rng.uniform(0.0, math.pi, COMPONENTS)}


def _host_points(mix, n, rng):
    """n mixture points on the host (places, query centres, cell seeds)."""
    k = rng.choice(COMPONENTS, size=n, p=mix["w"])
    u, v = (rng.standard_normal(n) * mix["s"][k, a] for a in (0, 1))
    co, si = np.cos(mix["th"][k]), np.sin(mix["th"][k])
    x, y = mix["c"][k, 0] + co * u - si * v, mix["c"][k, 1] + si * u + co * v
    out = (x < 0) | (x >= EXTENT) | (y < 0) | (y >= EXTENT)
    x[out], y[out] = mix["c"][k[out], 0], mix["c"][k[out], 1]
    return x, y


def _points(mix, n, seed):
    """n points on the GPU (float64 x and y), in no spatial order: mixture
    points inside the extent, or uniform ones in [0, 1)^2 without a mixture."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    kw = {"device": "cuda", "dtype": torch.float64}
    if mix is None:
        return torch.rand(n, generator=g, **kw), torch.rand(n, generator=g, **kw)
    cum = torch.tensor(np.cumsum(mix["w"])[:-1], **kw)
    co, si = np.cos(mix["th"]), np.sin(mix["th"])
    m = np.stack([mix["c"][:, 0], mix["c"][:, 1], co * mix["s"][:, 0], -si * mix["s"][:, 1], si * mix["s"][:, 0],
                  co * mix["s"][:, 1]])
    m = torch.tensor(m, **kw)
    x, y = torch.empty(n, **kw), torch.empty(n, **kw)
    for at in range(0, n, 1 << 24):
        todo = min(1 << 24, n - at)
        a, b = x[at:at + todo], y[at:at + todo]
        need = None
        for _ in range(8):   # points outside the extent are drawn again
            r = todo if need is None else need.numel()
            if r == 0:
                break
            k = torch.searchsorted(cum, torch.rand(r, generator=g, **kw))
            u, v = torch.randn(r, generator=g, **kw), torch.randn(r, generator=g, **kw)
            px = m[0][k] + m[2][k] * u + m[3][k] * v
            py = m[1][k] + m[4][k] * u + m[5][k] * v
            if need is None:
                a.copy_(px)
                b.copy_(py)
            else:
                a[need], b[need] = px, py
            need = ((a < 0) | (a >= EXTENT) | (b < 0) | (b >= EXTENT)).nonzero().squeeze(1)
        a.clamp_(0.0, math.nextafter(EXTENT, 0.0))
        b.clamp_(0.0, math.nextafter(EXTENT, 0.0))
    return x, y


def _csr(rings_x, rings_y, lengths):
    """A polygon set with one ring per polygon (or line)."""
    off = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    return {"n_polys": len(lengths), "poly_ring_off": None, "ring_vtx_off": off, "vx": rings_x, "vy": rings_y}


def _ranges(starts, lengths):
    """Concatenated aranges start .. start + length."""
    ends = np.cumsum(lengths)
    return np.arange(int(ends[-1])) - np.repeat(ends - lengths - starts, lengths)


def _tessellation(rng, mix, g, vmin, vmax, extent):
    """g x g cells tiling the extent: jittered nodes (cells small where the
    mixture is dense, when there is one), every side subdivided once with
    tapered jitter, so that neighbours share it bit for bit."""
    t = np.linspace(0.0, 1.0, g + 1)
    nx, ny = t * extent, t * extent
    if mix is not None:
        hx, hy = _host_points(mix, 20_000, rng)
        nx = 0.3 * nx + 0.7 * np.quantile(hx, t)
        ny = 0.3 * ny + 0.7 * np.quantile(hy, t)
        nx[[0, -1]] = ny[[0, -1]] = 0.0, extent
    X, Y = (a.copy() for a in np.meshgrid(nx, ny, indexing="ij"))
    dx, dy = np.diff(nx), np.diff(ny)
    rx, ry = np.minimum(dx[:-1], dx[1:])[:, None], np.minimum(dy[:-1], dy[1:])[None, :]
    if g > 1:
        X[1:-1, :] += 0.25 * rx * rng.uniform(-1, 1, (g - 1, g + 1))
        Y[:, 1:-1] += 0.25 * ry * rng.uniform(-1, 1, (g + 1, g - 1))
    # sides: horizontal (i, j)-(i + 1, j), then vertical (i, j)-(i, j + 1)
    ih, jh = (a.ravel() for a in np.meshgrid(np.arange(g), np.arange(g + 1), indexing="ij"))
    iv, jv = (a.ravel() for a in np.meshgrid(np.arange(g + 1), np.arange(g), indexing="ij"))
    ax, ay = np.concatenate([X[ih, jh], X[iv, jv]]), np.concatenate([Y[ih, jh], Y[iv, jv]])
    bx, by = np.concatenate([X[ih + 1, jh], X[iv, jv + 1]]), np.concatenate([Y[ih + 1, jh], Y[iv, jv + 1]])
    outer = np.concatenate([(jh == 0) | (jh == g), (iv == 0) | (iv == g)])
    # room across a side, so that the jitter of long thin cells never crosses
    room = np.concatenate([np.minimum(*(np.pad(dy, 1, mode="edge")[jh + k] for k in (0, 1))),
                           np.minimum(*(np.pad(dx, 1, mode="edge")[iv + k] for k in (0, 1)))])
    sub = rng.integers(max(0, vmin // 4 - 1), vmax // 4, size=ax.size)
    first = np.concatenate([[0], np.cumsum(sub)[:-1]])
    side = np.repeat(np.arange(ax.size), sub)
    f = (_ranges(np.zeros_like(sub), sub) + 1) / (sub[side] + 1)
    amp = 0.12 * np.sin(math.pi * f) * rng.uniform(-1, 1, f.size) * ~outer[side]
    ex, ey = bx - ax, by - ay
    amp *= np.minimum(1.0, room / np.hypot(ex, ey))[side]
    px, py = ax[side] + f * ex[side] - amp * ey[side], ay[side] + f * ey[side] + amp * ex[side]
    # rings: lower side, right side, upper side back, left side back
    ci, cj = (a.ravel() for a in np.meshgrid(np.arange(g), np.arange(g), indexing="ij"))
    nh = g * (g + 1)
    lo, up, le, ri = ci * (g + 1) + cj, ci * (g + 1) + cj + 1, nh + ci * g + cj, nh + (ci + 1) * g + cj
    length = 4 + sub[lo] + sub[ri] + sub[up] + sub[le]
    vx, vy = np.empty(int(length.sum())), np.empty(int(length.sum()))
    at = np.concatenate([[0], np.cumsum(length)[:-1]])
    for s, corner, back in ((lo, (ci, cj), False), (ri, (ci + 1, cj), False), (up, (ci + 1, cj + 1), True),
                            (le, (ci, cj + 1), True)):
        vx[at], vy[at] = X[corner], Y[corner]
        n = sub[s]
        k = _ranges(np.zeros_like(n), n) if n.sum() else np.zeros(0, dtype=np.int64)
        src = np.repeat(first[s], n) + (np.repeat(n, n) - 1 - k if back else k)
        vx[np.repeat(at + 1, n) + k], vy[np.repeat(at + 1, n) + k] = px[src], py[src]
        at = at + 1 + n
    return _csr(vx, vy, length)


def _stars(rng, nq, vmin, vmax, amin, amax, centres):
    """Star polygons: log-uniform vertex counts and areas, 30 % radius noise."""
    V = np.clip(np.floor(np.exp(rng.uniform(math.log(vmin), math.log(vmax + 1), nq))).astype(np.int64), vmin, vmax)
    R = np.sqrt(np.exp(rng.uniform(math.log(amin), math.log(amax), nq)) * EXTENT * EXTENT / math.pi)
    q = np.repeat(np.arange(nq), V)
    th = rng.uniform(0, 2 * math.pi, nq)[q] + 2 * math.pi * _ranges(np.zeros_like(V), V) / V[q]
    r = R[q] * (1.0 + 0.3 * rng.uniform(-1.0, 1.0, q.size))
    return _csr(centres[0][q] + r * np.cos(th), centres[1][q] + r * np.sin(th), V)


def _roads(rng, mix, nl, nv):
    """Road-like polylines: steps of about 150 m with a turning heading."""
    sx, sy = _host_points(mix, nl, rng)
    h = rng.uniform(0, 2 * math.pi, (nl, 1)) + np.cumsum(rng.normal(0.0, 0.35, (nl, nv - 1)), axis=1)
    st = 150.0 * rng.uniform(0.5, 1.5, (nl, nv - 1))
    xs = np.concatenate([sx[:, None], sx[:, None] + np.cumsum(st * np.cos(h), axis=1)], axis=1)
    ys = np.concatenate([sy[:, None], sy[:, None] + np.cumsum(st * np.sin(h), axis=1)], axis=1)
    return _csr(np.clip(xs, 0, EXTENT).ravel(), np.clip(ys, 0, EXTENT).ravel(), np.full(nl, nv, dtype=np.int64))


_contexts = {}


def _context(ppv):
    """One context per canvas resolution, kept as a program keeps it."""
    if ppv not in _contexts:
        ctx = spade.Context()
        ctx.set_pixels_per_vertex(ppv)
        _contexts[ppv] = ctx
    return _contexts[ppv]


class _Points(ctypes.Structure):
    """spade_points"""
    _fields_ = [("n", ctypes.c_int64), ("x", ctypes.c_void_p), ("y", ctypes.c_void_p)]


class _Disks(ctypes.Structure):
    """spade_disks"""
    _fields_ = [("n", ctypes.c_int64), ("cx", ctypes.c_void_p), ("cy", ctypes.c_void_p), ("r", ctypes.c_void_p),
                ("r_all", ctypes.c_double)]


_library = []


def _call(s, name, *args):
    """One call of the C library on the state's context."""
    if not _library:
        _library.append(ctypes.CDLL(spade.LIB_PATH))
        _library[0].spade_last_error.restype = ctypes.c_char_p
    rc = getattr(_library[0], name)(s["ctx"].handle, *args)
    if rc != 0:
        raise RuntimeError("%s: %d, %s" % (name, rc, _library[0].spade_last_error(s["ctx"].handle)))


def _ptr(t):
    return ctypes.c_void_p(t.data_ptr())


def _room(case):
    """Results that the program's output arrays hold: no result list of the
    case is longer (a star holds a few per cent of the points; the disks
    around evenly spread places hold a point 0.8 times on average)."""
    n, kind = int(case["points"]), case["kind"]
    if kind == "batch_select":
        return n * min(int(case["queries"]), math.ceil(1 + 0.15 * case["queries"]))
    if kind == "layered":
        return n * min(int(case["polygons"]), math.ceil(1 + 0.1 * case["polygons"]))
    if kind == "disk_join":
        return n * min(int(case["disks"]), 8)
    return n


def prepare(case, seed):
    rng = np.random.default_rng([int(seed), 17])
    kind, n = case["kind"], int(case["points"])
    ctx = _context(float(case.get("ppv", 96.0)))
    mix = None if case.get("law") == "uniform" else _mixture(rng)
    s = {"kind": kind, "ctx": ctx}
    x, y = _points(mix, n, int(seed))
    if kind in ("count", "pairs", "batch_count"):
        extent = 1.0 if mix is None else EXTENT
        cells = _tessellation(rng, mix if case["law"] == "census" else None, int(case["grid"]), int(case["vmin"]),
                              int(case["vmax"]), extent)
        if kind == "batch_count":
            s["table"] = ctx.table(x, y)
            s["batch"] = ctx.batch(ctx.polys(cells), [0, cells["n_polys"]])
            return s
        s["polys"] = ctx.polys(cells)
    elif kind == "select":
        centre = (np.array([EXTENT / 2]), np.array([EXTENT / 2]))
        v = int(case["vertices"])
        s["polys"] = ctx.polys(_stars(rng, 1, v, v, case["area"], case["area"], centre))
    elif kind in ("batch_select", "layered"):
        nq = int(case.get("queries") or case.get("polygons"))
        stars = _stars(rng, nq, int(case["vmin"]), int(case["vmax"]), case["amin"], case["amax"],
                       _host_points(mix, nq, rng))
        s["table"] = ctx.table(x, y)
        if kind == "layered":
            s["batch"] = ctx.layered(stars)
        else:
            s["polys"], s["bounds"] = ctx.polys(stars), np.arange(nq + 1, dtype=np.int64)
            s["batch"] = ctx.batch(s["polys"], s["bounds"])
            s["offsets"] = np.zeros(nq + 1, dtype=np.int64)
    elif kind == "disk_join":
        cx, cy = (torch.from_numpy(rng.uniform(0, EXTENT, int(case["disks"]))).cuda() for _ in range(2))
        s["places"] = cx, cy
        s["disks"] = _Disks(cx.numel(), cx.data_ptr(), cy.data_ptr(), None, float(case["radius"]))
    elif kind == "near_lines":
        s["lines"] = ctx.polys(_roads(rng, mix, int(case["lines"]), int(case["vertices"])))
        s["radius"] = float(case["radius"])
    else:
        px, py = _host_points(mix, 1, rng)
        s["px"], s["py"], s["k"] = float(px[0]), float(py[0]), int(case["k"])
    if kind not in ("batch_select", "layered"):
        s["x"], s["y"] = x, y
        s["points"] = _Points(n, x.data_ptr(), y.data_ptr())
    if kind not in ("count", "pairs", "knn"):
        s["room"] = _room(case)
        s["out"] = [torch.zeros(s["room"], dtype=torch.int32, device="cuda")
                    for _ in range(2 if kind in ("layered", "disk_join") else 1)]
    return s


def run(s):
    ctx, kind = s["ctx"], s["kind"]
    if kind == "count":
        return ctx.join_count(s["x"], s["y"], s["polys"])
    if kind == "pairs":
        return ctx.join_pairs(s["x"], s["y"], s["polys"])
    if kind == "batch_count":
        return ctx.batch_join_count(s["batch"], s["table"])
    if kind == "knn":
        return ctx.knn(s["x"], s["y"], s["px"], s["py"], s["k"])
    out, room, found = s["out"], ctypes.c_int64(s["room"]), ctypes.c_int64()
    if kind == "batch_select":
        ctx.batch(s["polys"], s["bounds"], into=s["batch"])
        _call(s, "spade_batch_select", s["batch"].handle, s["table"].handle, _ptr(out[0]), room,
              ctypes.c_void_p(s["offsets"].ctypes.data))
        return out[0], s["offsets"]
    if kind == "select":
        _call(s, "spade_select", ctypes.byref(s["points"]), ctypes.byref(s["polys"].cstruct()), _ptr(out[0]), room,
              ctypes.byref(found))
    elif kind == "layered":
        _call(s, "spade_batch_join_pairs", s["batch"].handle, s["table"].handle, _ptr(out[0]), _ptr(out[1]), room,
              ctypes.byref(found))
    elif kind == "disk_join":
        _call(s, "spade_distance_join_pairs", ctypes.byref(s["points"]), ctypes.byref(s["disks"]), _ptr(out[0]),
              _ptr(out[1]), room, ctypes.byref(found))
    else:
        _call(s, "spade_select_near_lines", ctypes.byref(s["points"]), ctypes.byref(s["lines"].cstruct()),
              ctypes.c_double(s["radius"]), _ptr(out[0]), room, ctypes.byref(found))
    return (*out, found.value)


def work(case):
    """Points and vertices read once (16 bytes each), results written once
    (their expected number: the data decide the real one)."""
    kind, n = case["kind"], int(case["points"])
    verts = (case.get("vmin", 0) + case.get("vmax", 0)) / 2
    if kind == "count":
        cells = case["grid"] ** 2
        b = 16 * n + cells * (16 * verts + 8)
    elif kind == "batch_count":
        b = 16 * n + 8 * case["grid"] ** 2          # the canvas set is resident
    elif kind == "pairs":
        b = 16 * n + 16 * verts * case["grid"] ** 2 + 8 * n    # a tessellation: one pair per point
    elif kind == "select":
        b = 16 * n + 16 * case["vertices"] + 4 * n * 1.5 * case["area"]
    elif kind in ("batch_select", "layered"):
        # areas log-uniform, points denser around the queries than on average
        nq = case.get("queries") or case.get("polygons")
        amin, amax = case["amin"], case["amax"]
        area = amin if amin == amax else (amax - amin) / math.log(amax / amin)
        found = n * nq * min(1.0, 2.0 * area)
        b = 16 * n + 16 * nq * verts / 3 + (4 if kind == "batch_select" else 8) * found
    elif kind == "disk_join":
        b = 16 * n + 16 * case["disks"] + 8 * n * case["disks"] * math.pi * case["radius"] ** 2 / EXTENT ** 2
    elif kind == "near_lines":
        b = 16 * n + 16 * case["lines"] * case["vertices"] + 4 * 0.3 * n
    else:
        b = 16 * n + 4 * case["k"]
    return {"bytes": float(b), "flops": 0.0}


def exact(case, seed):
    """Counts and ids are whole numbers: there is no rounded value to compare."""
    return None
