"""Performance cases: the work that programs have this library do, through
paper_2209_02878_amd.rsi, with seeded synthetic inputs made on the GPU.

listed() names the cases, draw(rng) gives one more from the same ranges.  A
case is a dict of plain values; its "kind" says which calls it stands for:

  query   Mesh.query_into / Mesh.query of segments against one mesh, with
          "rebuild" after the vertices have moved
  bary    first hits, then rsi_compact: the paper's compact `barycentric` outputs
  inside  Mesh.inside: the odd-parity test of points against a closed surface
  grad    rsi.first_hit and its gradients (vertices, both segment ends)
  batch   Batch.replay: the graph of rebuild + query over many meshes
  order   Mesh.segment_order: segments put into Morton order once

prepare(case, seed) makes the inputs, the tree and the output buffers,
run(state) is one pass, work(case) the traffic and arithmetic a pass cannot
do without, exact(case, seed) the floating outputs in 64 bits.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2209_02878_amd import rsi

DEVICE = "cuda"

# ------------------------------------------------------------- the cases --

# The ranges that the listed cases stand for and draw() covers.
TRIANGLES = (12, 500_000)
SEGMENTS = (32, 10_000_000)
MOST_PAIRS = 4.0e7  # segments x levels of the tree: a drawn case stays within the largest listed ones


def listed():
    return [
        # a pick or a probe bundle: a few rays at a time, the answer waited for by a user; launches are all of it
        {"name": "first_64seg_1922tri", "kind": "query", "surface": "heightfield", "triangles": 1_922, "segments": 64,
         "mode": "first", "alloc": True},
        # the smallest of the benchmark's workloads: visibility of 100k segments over a small terrain
        {"name": "bool_100kseg_1922tri", "kind": "query", "surface": "heightfield", "triangles": 1_922,
         "segments": 100_000, "mode": "bool"},
        # the paper's `intercept_count` at an ordinary, odd size, outputs allocated by the call
        {"name": "count_1Mseg_29768tri", "kind": "query", "surface": "heightfield", "triangles": 29_768,
         "segments": 1_000_003, "mode": "count", "alloc": True},
        # the benchmark's step: the terrain moved, 10M line-of-sight tests against the rebuilt tree
        {"name": "rebuild_bool_10Mseg_29768tri", "kind": "query", "surface": "heightfield", "triangles": 29_768,
         "segments": 10_000_000, "mode": "bool", "rebuild": True},
        # the benchmark's all-hits query: four slots per segment, the rest to the spill pool
        {"name": "all4_10Mseg_29768tri", "kind": "query", "surface": "heightfield", "triangles": 29_768,
         "segments": 10_000_000, "mode": "all", "capacity": 4},
        # every output of a large closed surface whose tree outgrows the L2
        {"name": "all4_first_10Mseg_499280tri", "kind": "query", "surface": "sphere", "triangles": 499_280,
         "segments": 10_000_000, "mode": "all|first|bool", "capacity": 4},
        # a depth image (640 x 480 rays) of a large surface that deforms from frame to frame
        {"name": "rebuild_first_307kseg_499280tri", "kind": "query", "surface": "sphere", "triangles": 499_280,
         "segments": 307_200, "mode": "first", "rebuild": True},
        # the paper's `barycentric` output of an ordinary, ragged number of segments
        {"name": "bary_3Mseg_29768tri", "kind": "bary", "surface": "heightfield", "triangles": 29_768,
         "segments": 2_999_999},
        # points of a volume grid classified against a closed surface
        {"name": "inside_4Mpt_499280tri", "kind": "inside", "surface": "sphere", "triangles": 499_280,
         "segments": 4_000_000},
        # one step of fitting a terrain to range data: refit, first hit, gradients
        {"name": "grad_4Mseg_199712tri", "kind": "grad", "surface": "heightfield", "triangles": 199_712,
         "segments": 4_000_000},
        # 64 moving meshes of very different sizes, each with its own segments, as one graph
        {"name": "batch64_bool", "kind": "batch", "meshes": 64, "tri_lo": 1_000, "tri_hi": 200_000, "seg_lo": 10_000,
         "seg_hi": 2_000_000, "mode": "bool"},
        # a training set's segments put in order before its first epoch
        {"name": "order_4Mseg", "kind": "order", "surface": "heightfield", "triangles": 29_768, "segments": 4_000_000},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["query"] * 6 + ["bary", "inside", "grad", "batch", "order"])
    if kind == "batch":
        meshes = _log_int(rng, 2, 64)
        tri_lo, seg_lo = _log_int(rng, 12, 2_000), _log_int(rng, 100, 20_000)
        return {"kind": "batch", "meshes": meshes, "tri_lo": tri_lo,
                "tri_hi": tri_lo * _log_int(rng, 2, 100), "seg_lo": seg_lo, "seg_hi": seg_lo * _log_int(rng, 2, 100),
                "mode": rng.choice(["bool", "bool", "first"])}
    surface = "sphere" if kind == "inside" else "heightfield" if kind == "grad" else rng.choice(["heightfield", "sphere"])
    triangles = _log_int(rng, *TRIANGLES)
    most = int(min(SEGMENTS[1], MOST_PAIRS / max(1.0, math.log(triangles, 4.0))))
    case = {"kind": kind, "surface": surface, "triangles": triangles}
    if kind == "query":
        case["segments"] = _log_int(rng, SEGMENTS[0], most)
        case["mode"] = rng.choice(["bool", "bool", "first", "first", "all", "all", "count", "all|first|bool", "first|bool"])
        if "all" in case["mode"]:
            case["capacity"] = rng.choice([1, 4, 4, 8, 16])
        case["rebuild"] = rng.random() < 0.4
        case["alloc"] = rng.random() < 0.4
        # options that programs set: larger leaves for less memory, the binary walk
        if rng.random() < 0.25:
            case["leaf_size"] = rng.choice([2, 4, 8])
        if rng.random() < 0.15:
            case["branching"] = 2
    else:
        case["segments"] = _log_int(rng, 1_000, min(most, 4_000_000) if kind == "grad" else most)
    return case


# ---------------------------------------------------------------- surfaces --

@functools.lru_cache(maxsize=32)
def _grid(n):
    """Triangles of an n x n vertex grid (vertex (i, j) is j * n + i)."""
    i, j = np.meshgrid(np.arange(n - 1), np.arange(n - 1), indexing="xy")
    v = (j * n + i).ravel()
    return np.stack([v, v + 1, v + n + 1, v, v + n + 1, v + n], 1).reshape(-1, 3).astype(np.int32)


@functools.lru_cache(maxsize=32)
def _geodesic(freq):
    """Unit geodesic sphere: each face of the icosahedron cut into freq^2
    triangles, outward winding, vertices on shared edges merged."""
    p = (1.0 + 5.0 ** 0.5) / 2.0
    iv = np.array([[-1, p, 0], [1, p, 0], [-1, -p, 0], [1, -p, 0], [0, -1, p], [0, 1, p], [0, -1, -p], [0, 1, -p],
                   [p, 0, -1], [p, 0, 1], [-p, 0, -1], [-p, 0, 1]], np.float64)
    iv /= np.linalg.norm(iv[0])
    d = np.linalg.norm(iv[:, None] - iv[None], axis=2)
    near = (d > 1e-9) & (d < d[d > 1e-9].min() * 1.01)
    faces = [(a, b, c) for a in range(12) for b in range(a + 1, 12) for c in range(b + 1, 12)
             if near[a, b] and near[b, c] and near[a, c]]
    a, b = np.meshgrid(np.arange(freq + 1), np.arange(freq + 1), indexing="ij")
    a, b = a[a + b <= freq], b[a + b <= freq]
    at = np.full((freq + 2, freq + 2), -1, np.int64)
    at[a, b] = np.arange(a.size)
    up = (a + b) < freq
    dn = (a + b) < freq - 1
    small = np.concatenate([np.stack([at[a[up], b[up]], at[a[up] + 1, b[up]], at[a[up], b[up] + 1]], 1),
                            np.stack([at[a[dn] + 1, b[dn]], at[a[dn] + 1, b[dn] + 1], at[a[dn], b[dn] + 1]], 1)])
    tag = np.random.RandomState(1).randint(1, 1 << 62, 12).astype(np.uint64)  # one key per lattice point
    keys, pts, tris = [], [], []
    for k, f in enumerate(faces):
        w = [freq - a - b, a, b]
        keys.append(sum(w[q].astype(np.uint64) * tag[f[q]] for q in range(3)))
        pts.append(sum(w[q][:, None] * iv[f[q]] for q in range(3)) / freq)
        tris.append(small + k * a.size)
    _, first, merged = np.unique(np.concatenate(keys), return_index=True, return_inverse=True)
    V = np.concatenate(pts)[first]
    V /= np.linalg.norm(V, axis=1, keepdims=True)
    T = merged.reshape(-1)[np.concatenate(tris)]
    x, y, z = V[T[:, 0]], V[T[:, 1]], V[T[:, 2]]
    turned = np.einsum("ij,ij->i", np.cross(y - x, z - x), x + y + z) < 0
    T[turned] = T[turned][:, [0, 2, 1]]
    return V, T.astype(np.int32)


def _noise(gen, q, octaves, base):
    """Lattice value noise at points q in [0, 1]^d (d 2 or 3), quintic fade."""
    dim, out = q.shape[1], torch.zeros(q.shape[0], dtype=torch.float64, device=q.device)
    for o in range(octaves):
        f = base << o
        lat = torch.rand((f + 1,) * dim, generator=gen, device=q.device, dtype=torch.float64).reshape(-1) * 2 - 1
        x = q.clamp(0, 1) * f
        i = x.floor().clamp(max=f - 1)
        w = x - i
        w = w * w * w * (w * (w * 6 - 15) + 10)
        i = i.long()
        for corner in range(1 << dim):
            idx, wt = torch.zeros_like(i[:, 0]), 2.0 ** -o
            for k in range(dim):
                up = corner >> k & 1
                idx = idx * (f + 1) + i[:, k] + up
                wt = wt * (w[:, k] if up else 1 - w[:, k])
            out += wt * lat[idx]
    return out


def _surface(kind, triangles, gen, jitter=0.1):
    """(V float32, T int32) on the GPU: a terrain over [0, 1]^2 with |z| up
    to 0.2 and xy jitter (in cells), or a closed star-shaped surface of radius
    1 +- 0.3."""
    if kind == "heightfield":
        n = _grid_side(triangles)
        g = torch.arange(n, device=DEVICE, dtype=torch.float64) / (n - 1)
        q = torch.stack([g.repeat(n), g.repeat_interleave(n)], 1)
        z = _noise(gen, q, 6, 4)
        z = z * (0.2 / z.abs().max().clamp(min=1e-9))
        off = (torch.rand(q.shape, generator=gen, device=DEVICE, dtype=torch.float64) * 2 - 1) * (jitter / (n - 1))
        return torch.cat([q + off, z[:, None]], 1).float(), torch.from_numpy(_grid(n)).to(DEVICE)
    U, T = _geodesic(_sphere_freq(triangles))
    U = torch.from_numpy(U).to(DEVICE)
    r = _noise(gen, U * 0.5 + 0.5, 4, 2)
    r = 1 + r * (0.3 / r.abs().max().clamp(min=1e-9))
    return (U * r[:, None]).float(), torch.from_numpy(T).to(DEVICE)


def _grid_side(triangles):
    return max(2, int(round(math.sqrt(triangles / 2.0))) + 1)


def _sphere_freq(triangles):
    return max(1, int(round(math.sqrt(triangles / 20.0))))


def _mesh_sizes(kind, triangles):
    """(vertices, triangles) of _surface()."""
    if kind == "heightfield":
        n = _grid_side(triangles)
        return n * n, 2 * (n - 1) * (n - 1)
    f = _sphere_freq(triangles)
    return 10 * f * f + 2, 20 * f * f


def _segments(kind, V, n, gen):
    """Terrain: starts uniform in the box, directions uniform, lengths
    log-uniform in [0.01, 1]; closed surface: both ends uniform in 1.5 times
    the box."""
    lo, hi = V.min(0).values, V.max(0).values
    u = torch.rand(n, 3, generator=gen, device=DEVICE)
    if kind == "heightfield":
        S = lo + u * (hi - lo)
        d = torch.randn(n, 3, generator=gen, device=DEVICE)
        d /= d.norm(dim=1, keepdim=True).clamp(min=1e-20)
        length = torch.exp(math.log(0.01) * torch.rand(n, 1, generator=gen, device=DEVICE))
        return S.contiguous(), (S + length * d).contiguous()
    c, h = 0.5 * (lo + hi), 0.75 * (hi - lo)
    w = torch.rand(n, 3, generator=gen, device=DEVICE)
    return (c + (2 * u - 1) * h).contiguous(), (c + (2 * w - 1) * h).contiguous()


def _vertical(n, gen):
    """Range data over a terrain: near-vertical segments from z = 1 to -1."""
    xy = 0.02 + 0.96 * torch.rand(n, 2, generator=gen, device=DEVICE)
    off = 0.01 * (2 * torch.rand(n, 2, generator=gen, device=DEVICE) - 1)
    one = torch.ones(n, 1, device=DEVICE)
    return torch.cat([xy, one], 1).contiguous(), torch.cat([xy + off, -one], 1).contiguous()


def _inputs(case, seed):
    """Everything of a single-mesh case that is drawn from the seed."""
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(int(seed))
    grad = case["kind"] == "grad"
    V, T = _surface(case["surface"], case["triangles"], gen, jitter=0.0 if grad else 0.1)
    n = case["segments"]
    if grad:
        S, E = _vertical(n, gen)
        up = [torch.randn(shape, generator=gen, device=DEVICE) for shape in ((n,), (n, 2), (n, 3))]
        return {"V": V, "T": T, "S": S, "E": E, "up": up}
    S, E = _segments(case["surface"], V, n, gen)
    return {"V": V, "T": T, "S": S, "E": E}


def _batch_sizes(case):
    """(surface, triangles, segments) of each mesh of a batch: sizes spread
    evenly over the logarithm of their ranges, paired without order."""
    golden, out = 0.6180339887498949, []
    for m in range(case["meshes"]):
        x, y = (m + 0.5) * golden % 1.0, (m + 0.5) * golden * golden * 7 % 1.0
        out.append(("heightfield" if m % 2 == 0 else "sphere",
                    int(case["tri_lo"] * (case["tri_hi"] / case["tri_lo"]) ** x),
                    int(case["seg_lo"] * (case["seg_hi"] / case["seg_lo"]) ** y)))
    return out


# ------------------------------------------------------------- one pass ----

_OUT = {"hit": (torch.uint8, 1), "tri": (torch.int32, 1), "t": (torch.float32, 1), "uv": (torch.float32, 2),
        "point": (torch.float32, 3)}


def prepare(case, seed):
    if case["kind"] == "batch":
        return _prepare_batch(case, seed)
    st = _inputs(case, seed)
    st["case"] = case
    st["mesh"] = rsi.Mesh(st["V"], st["T"], leaf_size=case.get("leaf_size", 0), branching=case.get("branching", 0))
    if case["kind"] == "query" and not case.get("alloc"):
        st["out"] = st["mesh"].alloc_outputs(case["segments"], case["mode"], case.get("capacity", 4))
    if case["kind"] == "bary":
        n = case["segments"]
        st["out"] = st["mesh"].alloc_outputs(n, "first")
        st["rows"] = {"ids": torch.zeros(n, dtype=torch.int32, device=DEVICE),
                      "dist": torch.zeros(n, device=DEVICE),
                      "tri_out": torch.zeros(n, dtype=torch.int32, device=DEVICE),
                      "point_out": torch.zeros(n, 3, device=DEVICE)}
    if case.get("rebuild"):  # the vertices after the surface has moved
        st["V"] = (st["V"] + 0.01 * torch.sin(7.0 * st["V"].roll(1, 1))).contiguous()
    if case["kind"] == "grad":
        for k in ("V", "S", "E"):
            st[k].requires_grad_(True)
    if case["kind"] == "query" and "all" in case["mode"]:
        # the library's spill pool grows to fit once, as rsi_query_stats asks
        st["mesh"].query(st["S"], st["E"], case["mode"], case.get("capacity", 4))
    return st


def _prepare_batch(case, seed):
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(int(seed))
    meshes, segs = [], []
    for kind, nt, ns in _batch_sizes(case):
        V, T = _surface(kind, nt, gen, jitter=0.25)
        meshes.append((V, T))
        segs.append(_segments(kind, V, ns, gen))
    total = sum(S.shape[0] for S, _ in segs)
    names = ["hit"] if case["mode"] == "bool" else ["tri", "t", "uv", "point"]
    whole = {k: torch.empty((total, _OUT[k][1]) if _OUT[k][1] > 1 else (total,), dtype=_OUT[k][0], device=DEVICE)
             for k in names}
    outs, at = [], 0
    for S, _ in segs:
        outs.append({k: whole[k][at:at + S.shape[0]] for k in names})
        at += S.shape[0]
    batch = rsi.Batch(meshes)
    batch.capture(segs, case["mode"], outs, rebuild=True)
    return {"case": case, "batch": batch, "whole": whole, "keep": (meshes, segs, outs)}


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "batch":
        st["batch"].replay()
        return st["whole"]
    mesh, S, E = st["mesh"], st["S"], st["E"]
    if kind == "query":
        if case.get("rebuild"):
            mesh.rebuild(st["V"], st["T"])
        if not case.get("alloc"):
            return mesh.query_into(S, E, case["mode"], st["out"], case.get("capacity", 4))
        out = mesh.query(S, E, case["mode"], case.get("capacity", 4))
        out.pop("spill", None)  # the pool's lists, whose order is unspecified
        return out
    if kind == "bary":
        r, rows = mesh.query_into(S, E, "first", st["out"]), st["rows"]
        k = rsi.rsi_compact(mesh.handle, case["segments"], tri=r["tri"], t=r["t"], point=r["point"], S=S, E=E, **rows)
        return {"rows": k, **rows}  # the first k rows of each
    if kind == "inside":
        return mesh.inside(S)
    if kind == "grad":
        t, uv, point, tri = rsi.first_hit(st["V"], S, E, mesh)
        dV, dS, dE = torch.autograd.grad([t, uv, point], [st["V"], S, E], st["up"])
        return {"t": t, "uv": uv, "point": point, "tri": tri, "dV": dV, "dS": dS, "dE": dE}
    return mesh.segment_order(S, E)


def _walk_flops(n_r, n_t):
    # one path down a four-way tree, four box tests (25 operations) per
    # level, and one triangle test (50)
    return n_r * (100.0 * max(1.0, math.ceil(math.log(max(n_t, 2), 4.0))) + 50.0)


def work(case):
    if case["kind"] == "batch":
        b = f = 0.0
        for kind, nt, ns in _batch_sizes(case):
            n_v, n_t = _mesh_sizes(kind, nt)
            b += 12.0 * n_v + 12.0 * n_t + ns * (24.0 + (1.0 if case["mode"] == "bool" else 28.0))
            f += _walk_flops(ns, n_t)
        return {"bytes": b, "flops": f}
    n_v, n_t = _mesh_sizes(case["surface"], case["triangles"])
    n, mesh = float(case["segments"]), 12.0 * n_v + 12.0 * n_t
    kind = case["kind"]
    if kind == "order":  # both ends and the order out, then gathered
        return {"bytes": n * (24.0 + 4.0 + 24.0), "flops": n * 30.0}
    if kind == "inside":  # point in, far end, count and flag out
        return {"bytes": mesh + n * (12.0 + 12.0 + 4.0 + 1.0), "flops": _walk_flops(n, n_t)}
    if kind == "bary":  # at most one compact row per segment; about a fifth of them cross
        return {"bytes": mesh + n * 24.0 + 0.2 * n * 24.0, "flops": _walk_flops(n, n_t)}
    if kind == "grad":  # forward, then upstream gradients in, three gradients out
        return {"bytes": mesh + 12.0 * n_v + n * (24.0 + 28.0 + 24.0 + 24.0 + 4.0 + 24.0),
                "flops": _walk_flops(n, n_t) + 150.0 * n}
    per = 24.0
    modes = case["mode"].split("|")
    per += 1.0 if "bool" in modes else 0.0
    per += 28.0 if "first" in modes else 0.0
    per += 4.0 if "count" in modes else 0.0
    per += 4.0 + 8.0 * case.get("capacity", 4) if "all" in modes else 0.0
    return {"bytes": mesh + n * per, "flops": _walk_flops(n, n_t)}


# ------------------------------------------------- the values in 64 bits ---

def _tree64(V, T):
    """Boxes over the triangles in Morton order, eight to one per level, from
    the leaves up: [(lo, hi)] per level, and the triangles' order."""
    P = V.double()[T.long()]
    c = P.mean(1)
    lo, hi = c.min(0).values, c.max(0).values
    q = ((c - lo) / (hi - lo).clamp(min=1e-30) * 1023).long()
    key = torch.zeros_like(q[:, 0])
    for bit in range(10):
        for k in range(3):
            key |= (q[:, k] >> bit & 1) << (3 * bit + k)
    order = key.argsort(stable=True)
    lo, hi = P[order].min(1).values, P[order].max(1).values
    pad = 1e-9 * float((hi.max(0).values - lo.min(0).values).max())
    levels = [(lo - pad, hi + pad)]
    while levels[-1][0].shape[0] > 8:
        lo, hi = levels[-1]
        m = -(-lo.shape[0] // 8) * 8 - lo.shape[0]
        if m:
            lo = torch.cat([lo, lo[-1:].expand(m, 3)])
            hi = torch.cat([hi, hi[-1:].expand(m, 3)])
        levels.append((lo.reshape(-1, 8, 3).min(1).values, hi.reshape(-1, 8, 3).max(1).values))
    return levels, order


def _crossings64(V, T, S, E):
    """Every crossing of the segments (S, E) and the triangles in 64 bits,
    closed at every boundary: (segment, t, u, v) ordered by (segment, t)."""
    levels, order = _tree64(V, T)
    P = V.double()[T.long()[order]]
    v0, e1, e2 = P[:, 0], P[:, 1] - P[:, 0], P[:, 2] - P[:, 0]
    found, step = [], 250_000
    for at in range(0, S.shape[0], step):
        o = S[at:at + step].double()
        d = E[at:at + step].double() - o
        inv = 1.0 / torch.where(d.abs() < 1e-30, torch.full_like(d, 1e-30), d)
        top = levels[-1][0].shape[0]
        seg = torch.arange(o.shape[0], device=o.device).repeat_interleave(top)
        node = torch.arange(top, device=o.device).repeat(o.shape[0])
        for k in range(len(levels) - 1, -1, -1):
            lo, hi = levels[k]
            a, b = (lo[node] - o[seg]) * inv[seg], (hi[node] - o[seg]) * inv[seg]
            near = torch.minimum(a, b).amax(1).clamp(min=0)
            far = torch.maximum(a, b).amin(1).clamp(max=1)
            keep = near <= far * (1 + 1e-9) + 1e-12
            seg, node = seg[keep], node[keep]
            if k:
                seg = seg.repeat_interleave(8)
                node = (8 * node[:, None] + torch.arange(8, device=o.device)).reshape(-1)
                inside = node < levels[k - 1][0].shape[0]
                seg, node = seg[inside], node[inside]
        dd, q = d[seg], o[seg] - v0[node]
        p = torch.cross(dd, e2[node], dim=1)
        r = torch.cross(q, e1[node], dim=1)
        det = (e1[node] * p).sum(1)
        u, v, t = ((q * p).sum(1) / det, (dd * r).sum(1) / det, (e2[node] * r).sum(1) / det)
        ok = (det != 0) & (u >= 0) & (v >= 0) & (u + v <= 1) & (t >= 0) & (t <= 1)
        found.append([seg[ok] + at, t[ok], u[ok], v[ok], order[node[ok]]])
    seg, t, u, v, tri = (torch.cat(x) for x in zip(*found))
    by = t.argsort(stable=True)
    by = by[seg[by].argsort(stable=True)]
    return seg[by], t[by], u[by], v[by], tri[by]


def _first64(st, n):
    seg, t, u, v, tri = _crossings64(st["V"], st["T"], st["S"], st["E"])
    head = torch.ones_like(seg, dtype=torch.bool)
    head[1:] = seg[1:] != seg[:-1]
    seg, t, u, v, tri = seg[head], t[head], u[head], v[head], tri[head]
    full = torch.full((n,), math.inf, dtype=torch.float64, device=t.device)
    full[seg] = t
    uv = torch.zeros(n, 2, dtype=torch.float64, device=t.device)
    uv[seg] = torch.stack([u, v], 1)
    o, e = st["S"].double()[seg], st["E"].double()[seg]
    point = torch.zeros(n, 3, dtype=torch.float64, device=t.device)
    point[seg] = o + t[:, None] * (e - o)
    return {"t": full, "uv": uv, "point": point}, seg, tri


def _slots64(st, n, capacity):
    seg, t, _, _, _ = _crossings64(st["V"], st["T"], st["S"], st["E"])
    count = torch.bincount(seg, minlength=n)
    rank = torch.arange(seg.numel(), device=seg.device) - (count.cumsum(0) - count)[seg]
    ts = torch.full((n, capacity), math.inf, dtype=torch.float64, device=t.device)
    keep = rank < capacity
    ts[seg[keep], rank[keep]] = t[keep]
    return ts


def _inside64(st):
    P = st["S"].double()
    used = st["V"][st["T"].long().reshape(-1)].double()
    lo, hi = used.min(0).values, used.max(0).values
    c, R = 0.5 * (lo + hi), 0.5 * (hi - lo).norm()
    u = torch.tensor([0.515216053, 0.352064312, 0.781410992], dtype=torch.float32, device=P.device).double()
    return P + ((P - c).norm(dim=1, keepdim=True) + 2 * R + 1) * u


def _gradients64(st, seg, tri):
    """Gradients of sum(up . (t, u, v, P)) over the hit segments."""
    V, S, E = (st[k].detach().double().requires_grad_(True) for k in ("V", "S", "E"))
    P = V[st["T"].long()[tri]]
    v0, e1, e2 = P[:, 0], P[:, 1] - P[:, 0], P[:, 2] - P[:, 0]
    o, d = S[seg], E[seg] - S[seg]
    p = torch.cross(d, e2, dim=1)
    q = o - v0
    r = torch.cross(q, e1, dim=1)
    det = (e1 * p).sum(1)
    t, u, v = (e2 * r).sum(1) / det, (q * p).sum(1) / det, (d * r).sum(1) / det
    gt, guv, gp = (g.double()[seg] for g in st["up"])
    loss = (gt * t).sum() + (guv[:, 0] * u).sum() + (guv[:, 1] * v).sum() + (gp * (o + t[:, None] * d)).sum()
    return torch.autograd.grad(loss, [V, S, E])


def exact(case, seed):
    kind = case["kind"]
    if kind in ("batch", "order"):
        return None  # flags, or the inputs themselves in another order
    st = _inputs(case, seed)
    n = case["segments"]
    if case.get("rebuild"):
        st["V"] = (st["V"] + 0.01 * torch.sin(7.0 * st["V"].roll(1, 1))).contiguous()
    if kind == "inside":
        return {"E": _inside64(st), "count": None, "inside": None}
    if kind == "bary":
        out, seg, _ = _first64(st, n)
        length = (st["E"].double() - st["S"].double()).norm(dim=1)[seg]
        dist, point = torch.zeros_like(out["t"]), torch.zeros_like(out["point"])
        dist[:seg.numel()], point[:seg.numel()] = out["t"][seg] * length, out["point"][seg]
        return {"dist": dist, "point_out": point, "ids": None, "tri_out": None, "rows": None}
    if kind == "grad":
        out, seg, tri = _first64(st, n)
        dV, dS, dE = _gradients64(st, seg, tri)
        return {**out, "dV": dV, "dS": dS, "dE": dE, "tri": None}
    modes, out = case["mode"].split("|"), {}
    if "first" in modes:
        out.update(_first64(st, n)[0])
    if "all" in modes:
        out["ts"] = _slots64(st, n, case.get("capacity", 4))
    return out or None
