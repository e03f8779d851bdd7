"""Workloads that the speed of this library is measured on.

Every case is one call (or one forward and backward) through the public
Python API on inputs made on the GPU from a seed: triangle soups and
tetrahedral soups whose private vertices have to be merged again, meshes that
are already indexed, the paper's quad grid in stored order, packed batches,
mesh merging, sub-mesh extraction and the attribute gather. Sizes run from a
few hundred vertices to the 26.4M-vertex soup of the benchmark.

  listed()          the named cases
  draw(rng)         one more case of the same ranges
  prepare(case, s)  inputs, outputs and workspace a program holds before the call
  run(state)        one pass; returns every output
  work(case)        bytes and operations no implementation can do without
  exact(case, s)    the same outputs from plain torch in 64 bits
"""
import math

import torch

import paper_2109_09812_amd as mrx

# Words per vertex record that meshes come with: positions (2 or 3 words),
# with texture coordinates, normals or both, and full sets of attributes.
WIDTHS = (2, 3, 3, 3, 4, 5, 6, 8, 8, 11, 12, 16)

# Corners (a, b, c) of the five tetrahedra a cube is split into.
_TETS = (((0, 0, 0), (1, 0, 0), (0, 1, 0), (0, 0, 1)), ((1, 1, 0), (1, 0, 0), (0, 1, 0), (1, 1, 1)),
         ((1, 0, 1), (1, 0, 0), (0, 0, 1), (1, 1, 1)), ((0, 1, 1), (0, 1, 0), (0, 0, 1), (1, 1, 1)),
         ((1, 0, 0), (0, 1, 0), (0, 0, 1), (1, 1, 1)))


def listed():
    return [
        # one small object, re-indexed by a plain call: latency
        {"name": "soup16", "kind": "soup", "nx": 16, "ny": 16, "words": 3, "unused": 0.1, "call": "api"},
        # a small part inside a loop that keeps its buffers
        {"name": "soup57x61", "kind": "soup", "nx": 57, "ny": 61, "words": 3, "unused": 0.05, "call": "launch"},
        # an ordinary scanned object, plain call with trimmed outputs
        {"name": "soup256", "kind": "soup", "nx": 255, "ny": 255, "words": 3, "unused": 0.1, "call": "api"},
        # the benchmark's soup: 26.4M vertices
        {"name": "soup2048", "kind": "soup", "nx": 2047, "ny": 2047, "words": 3, "unused": 0.05, "call": "launch"},
        # volume mesh with position, normal and texture coordinates per vertex (32-byte records)
        {"name": "tets64", "kind": "tets", "n": 64, "unused": 0.03, "call": "launch"},
        # the paper's own grid: 8-byte records in stored order, every fifth vertex unused
        {"name": "quads1024", "kind": "quads", "n": 1024, "call": "launch"},
        # a mesh that is already indexed, after a cut that left some vertices unused
        {"name": "indexed1000", "kind": "indexed", "nx": 999, "ny": 1001, "words": 6, "unused": 0.1, "call": "launch"},
        # a scene of independent objects in one call, sizes as in the batched benchmark
        {"name": "batch256", "kind": "batch", "meshes": 256, "lo": 100, "hi": 200000, "call": "launch"},
        # thousands of small parts
        {"name": "parts4096", "kind": "batch", "meshes": 4096, "lo": 20, "hi": 400, "call": "api"},
        # tiles of one surface merged into a single mesh, borders shared
        {"name": "merge64", "kind": "merge", "tiles": 8, "quads": 120, "call": "launch"},
        # half of a soup's triangles kept (kept buffers: how many outputs there are is known on the device alone)
        {"name": "extract1024", "kind": "extract", "nx": 1023, "ny": 1023, "words": 3, "unused": 0.05, "keep": 0.5,
         "call": "launch"},
        # per-vertex features through the new -> old map, forward and backward
        {"name": "gather10M", "kind": "gather", "old": 10_000_000, "new": 1_602_531, "channels": 16, "double": False,
         "injective": True, "validate": False},
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["soup", "soup", "soup", "tets", "quads", "indexed", "batch", "merge", "extract", "gather"])
    call = rng.choice(["api", "launch"])
    words = rng.choice(WIDTHS)
    # a soup of nx x ny quads has 6.3 vertices per quad: wide records stay below the largest listed case
    most = 2000 * 2000 * 3 / max(3, words)
    unused = round(rng.uniform(0.0, 0.3), 3)
    if kind in ("soup", "extract", "indexed"):
        quads = _logint(rng, 30, most)
        nx = max(1, int(round(math.sqrt(quads) * math.exp(rng.uniform(-0.7, 0.7)))))
        case = {"kind": kind, "nx": nx, "ny": max(1, quads // nx), "words": words, "unused": unused, "call": call}
        if kind == "extract":
            case.update(keep=round(rng.uniform(0.05, 0.95), 3), call="launch")
        return case
    if kind == "tets":
        return {"kind": kind, "n": _logint(rng, 2, 72), "unused": unused, "call": call}
    if kind == "quads":
        return {"kind": kind, "n": _logint(rng, 6, 1800), "call": call}
    if kind == "batch":
        hi = _logint(rng, 200, 200000)
        meshes = max(2, min(_logint(rng, 2, 5000), int(2.5e7 / hi)))
        return {"kind": kind, "meshes": meshes, "lo": rng.randint(1, 100), "hi": hi, "call": call}
    if kind == "merge":
        tiles = rng.randint(2, 12)
        return {"kind": kind, "tiles": tiles, "quads": _logint(rng, 5, 1500 / tiles), "call": call}
    old = _logint(rng, 1000, 12_000_000)
    return {"kind": kind, "old": old, "new": max(1, int(old * rng.uniform(0.1, 0.9))),
            "channels": rng.choice([1, 2, 3, 4, 7, 8, 13, 16]), "double": rng.random() < 0.25,
            "injective": rng.random() < 0.7, "validate": rng.random() < 0.5}


# ------------------------------------------------------------------ inputs


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(2109_09812 + 7919 * int(seed))


def _points(i, j, sx, sy, words):
    """Grid point records: x, y, a height, then attributes that follow from
    the position (normal, texture coordinates, colours)."""
    x = i.to(torch.float32) / sx
    y = j.to(torch.float32) / sy
    z = ((31 * i + 17 * j) % 1024).to(torch.float32) / 1024
    cols = [x, y, z, x - 0.5, 0.5 - y, z * 0.25, x * y, 1 - x, 1 - y, x + z, y + z, x - z, y - z, x * z, y * z, z - 0.5]
    return torch.stack(cols[:words], dim=1)


def _shuffled(vtx, unused, gen):
    """`vtx` with that fraction of random records appended, permuted; the
    place of every original row in the result."""
    n0, k = vtx.shape
    extra = torch.rand((int(unused * n0), k), generator=gen, device="cuda")
    vtx = torch.cat([vtx, extra])
    perm = torch.randperm(vtx.shape[0], generator=gen, device="cuda")
    where = torch.empty_like(perm)
    where[perm] = torch.arange(perm.numel(), device="cuda")
    return vtx[perm].contiguous(), where[:n0]


def _soup_corners(nx, ny):
    """(i, j) of the corners of an nx x ny quad patch's triangles, two per quad."""
    q = torch.arange(nx * ny, device="cuda")
    qi, qj = q % nx, q // nx
    di = torch.tensor([0, 1, 1, 0, 1, 0], device="cuda")
    dj = torch.tensor([0, 0, 1, 0, 1, 1], device="cuda")
    return (qi[:, None] + di).reshape(-1), (qj[:, None] + dj).reshape(-1)


def _origin(seed):
    return int(seed) % 61


def _soup(case, seed, gen):
    i, j = _soup_corners(case["nx"], case["ny"])
    pts = _points(i + _origin(seed), j, case["nx"], case["ny"], case["words"])
    vtx, where = _shuffled(pts, case["unused"], gen)
    return vtx, where.to(torch.int32).view(-1, 3).contiguous()


def _tets(case, seed, gen):
    n = case["n"]
    c = torch.arange(n ** 3, device="cuda")
    cells = torch.stack([c // (n * n) + _origin(seed), c // n % n, c % n], dim=1)
    corners = torch.tensor(_TETS, device="cuda").view(1, 20, 3)
    p = (cells[:, None] + corners).reshape(-1, 3).to(torch.float32) / n
    d = p - torch.tensor([0.5, 0.5, -1.0], device="cuda")
    d = d / (d * d).sum(dim=1, keepdim=True).sqrt()
    vtx, where = _shuffled(torch.cat([p, d, p[:, :2]], dim=1), case["unused"], gen)
    return vtx, where.to(torch.int32).view(-1, 4).contiguous()


def _quads(case, seed, gen):
    n = case["n"]
    q = torch.arange(n * n, device="cuda")
    d = torch.tensor([[0, 0], [1, 0], [1, 1], [0, 1], [0.5, 0.5]], device="cuda")
    at = torch.stack([q % n + _origin(seed), q // n], dim=1).to(torch.float32)
    vtx = ((at[:, None] + d) / n).reshape(-1, 2).contiguous()
    idx = 5 * q[:, None] + torch.arange(4, device="cuda")
    return vtx, idx.to(torch.int32).contiguous()


def _indexed(case, seed, gen):
    nx, ny = case["nx"], case["ny"]
    v = torch.arange((nx + 1) * (ny + 1), device="cuda")
    vtx = _points(v % (nx + 1) + _origin(seed), v // (nx + 1), nx, ny, case["words"]).contiguous()
    i, j = _soup_corners(nx, ny)
    tris = (j * (nx + 1) + i).view(-1, 3)
    # a band of the surface is cut away: its vertices stay in the array, unused
    tris = tris[: max(1, int(tris.shape[0] * (1 - case["unused"])))]
    return vtx, tris.to(torch.int32).contiguous()


def _ragged_soups(sizes, seed, gen):
    """Independent soup patches of sizes[b] triangles, packed; 5% unused each,
    each mesh's vertices permuted within the mesh."""
    t = sizes
    extra = (t * 3) // 20
    nb = 3 * t + extra
    vo = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"), nb.cumsum(0)])
    eo = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"), t.cumsum(0)])
    n, e, b = int(vo[-1]), int(eo[-1]), t.numel()
    width = ((t + 1) // 2).to(torch.float64).sqrt().ceil().to(torch.int64).clamp(min=1)
    mesh_v = torch.repeat_interleave(torch.arange(b, device="cuda"), nb)
    local = torch.arange(n, device="cuda") - vo[mesh_v]
    w = width[mesh_v]
    tri, corner = local // 3, local % 3 + 3 * (local // 3 % 2)
    quad = tri // 2
    di = torch.tensor([0, 1, 1, 0, 1, 0], device="cuda")[corner]
    dj = torch.tensor([0, 0, 1, 0, 1, 1], device="cuda")[corner]
    i, j = quad % w + di, quad // w + dj
    vtx = torch.stack([(i + _origin(seed)).to(torch.float32) / w, j.to(torch.float32) / w,
                       ((31 * i + 17 * j) % 1024).to(torch.float32) / 1024], dim=1)
    spare = local >= 3 * t[mesh_v]
    vtx = torch.where(spare[:, None], torch.rand((n, 3), generator=gen, device="cuda"), vtx)
    perm = torch.randperm(n, generator=gen, device="cuda")
    perm = perm[torch.sort(mesh_v[perm], stable=True).indices]  # a random order inside every mesh
    where = torch.empty_like(perm)
    where[perm] = torch.arange(n, device="cuda")
    mesh_e = torch.repeat_interleave(torch.arange(b, device="cuda"), t)
    first = vo[mesh_e] + 3 * (torch.arange(e, device="cuda") - eo[mesh_e])
    idx = where[first[:, None] + torch.arange(3, device="cuda")] - vo[mesh_e][:, None]
    return vtx[perm].contiguous(), vo, idx.to(torch.int32).contiguous(), eo


def _batch_sizes(case, seed):
    """Triangles per mesh, log-uniform in [lo, hi]: stratified, in a seeded
    order, so that a case has the same total with every seed."""
    b = case["meshes"]
    u = (torch.arange(b, dtype=torch.float64) + 0.5) / b
    t = torch.exp(math.log(case["lo"]) + u * (math.log(case["hi"]) - math.log(case["lo"]))).round().to(torch.int64)
    g = torch.Generator().manual_seed(int(seed))
    return t.clamp(min=1)[torch.randperm(b, generator=g)]


def _tiles(case, seed, gen):
    """tiles x tiles soup patches of one surface, each a mesh of its own."""
    q, tl = case["quads"], case["tiles"]
    i, j = _soup_corners(q, q)
    ti = torch.arange(tl * tl, device="cuda")
    gi = (ti[:, None] % tl * q + i).reshape(-1) + _origin(seed)
    gj = (ti[:, None] // tl * q + j).reshape(-1)
    vtx = _points(gi, gj, tl * q, tl * q, 3)
    per = i.numel()
    perm = torch.rand((tl * tl, per), generator=gen, device="cuda").argsort(dim=1)
    where = torch.empty_like(perm)
    where.scatter_(1, perm, torch.arange(per, device="cuda").expand(tl * tl, per).contiguous())
    vtx = vtx.view(tl * tl, per, 3).gather(1, perm[..., None].expand(-1, -1, 3)).reshape(-1, 3)
    vo = torch.arange(tl * tl + 1, device="cuda") * per
    return vtx.contiguous(), vo, where.to(torch.int32).view(-1, 3).contiguous(), vo // 3


_SINGLE = {"soup": _soup, "tets": _tets, "quads": _quads, "indexed": _indexed, "extract": _soup}


def _inputs(case, seed):
    gen = _gen(seed)
    kind = case["kind"]
    if kind in _SINGLE:
        vtx, idx = _SINGLE[kind](case, seed, gen)
        s = {"vtx": vtx, "idx": idx}
        if kind == "extract":
            s["keep"] = torch.rand(idx.shape[0], generator=gen, device="cuda") < case["keep"]
        return s
    if kind == "batch":
        names = ("vtx", "vtx_offsets", "idx", "elem_offsets")
        return dict(zip(names, _ragged_soups(_batch_sizes(case, seed).to("cuda"), seed, gen)))
    if kind == "merge":
        return dict(zip(("vtx", "vtx_offsets", "idx", "elem_offsets"), _tiles(case, seed, gen)))
    dtype = torch.float64 if case["double"] else torch.float32
    attrs = torch.randn((case["old"], case["channels"]), generator=gen, device="cuda", dtype=dtype)
    grad = torch.randn((case["new"], case["channels"]), generator=gen, device="cuda", dtype=dtype)
    if case["injective"]:
        new2old = torch.randperm(case["old"], generator=gen, device="cuda")[: case["new"]]
    else:
        new2old = torch.randint(0, case["old"], (case["new"],), generator=gen, device="cuda")
    return {"attrs": attrs, "grad": grad, "new2old": new2old.to(torch.int32)}


def prepare(case, seed):
    s = dict(_inputs(case, seed), case=case)
    kind = case["kind"]
    if kind == "gather":
        s["attrs"].requires_grad_(True)
    elif case["call"] == "launch":
        if kind == "batch":
            r = mrx.BatchedReindexer(s["vtx"], s["vtx_offsets"], s["idx"], s["elem_offsets"])
        elif kind == "merge":
            r = mrx.MeshMerger(s["vtx"], s["vtx_offsets"], s["idx"], s["elem_offsets"])
        elif kind == "extract":
            r = mrx.SubmeshExtractor(s["vtx"], s["idx"], s["keep"])
        else:
            r = mrx.Reindexer(s["vtx"], s["idx"])
        # capacity beyond the outputs is never written: give it a value
        for t in (r.out_vtx, r.out_idx, r.new2old):
            t.zero_()
        s["plan"] = r
    return s


# --------------------------------------------------------------------- run


def run(s):
    case, kind = s["case"], s["case"]["kind"]
    if kind == "gather":
        a = s["attrs"]
        a.grad = None
        out = mrx.gather_attrs(a, s["new2old"], case["injective"], case["validate"])
        out.backward(s["grad"])
        return {"out": out.detach(), "grad": a.grad}
    if case["call"] == "launch":
        r = s["plan"]
        r.launch()
    elif kind == "batch":
        r = mrx.reindex_mesh_batched(s["vtx"], s["vtx_offsets"], s["idx"], s["elem_offsets"])
    elif kind == "merge":
        r = mrx.merge_meshes(s["vtx"], s["vtx_offsets"], s["idx"], s["elem_offsets"])
    else:
        r = mrx.reindex_mesh(s["vtx"], s["idx"])
    out = {"vtx": r.out_vtx, "idx": r.out_idx, "old2new": r.old2new, "new2old": r.new2old}
    if kind == "batch":
        out["offsets"] = r.out_vtx_offsets
    else:
        out["meta"] = r.meta
    return out


# -------------------------------------------------------------------- work


def _sizes(case):
    """Vertices, index entries, output vertices, record words of a case."""
    kind = case["kind"]
    if kind in ("soup", "extract"):
        n0 = 6 * case["nx"] * case["ny"]
        return n0 + int(case["unused"] * n0), n0, (case["nx"] + 1) * (case["ny"] + 1), case["words"]
    if kind == "tets":
        n0 = 20 * case["n"] ** 3
        return n0 + int(case["unused"] * n0), n0, (case["n"] + 1) ** 3, 8
    if kind == "quads":
        return 5 * case["n"] ** 2, 4 * case["n"] ** 2, (case["n"] + 1) ** 2, 2
    if kind == "indexed":
        n = (case["nx"] + 1) * (case["ny"] + 1)
        return n, int(6 * case["nx"] * case["ny"] * (1 - case["unused"])), int(n * (1 - case["unused"])), case["words"]
    if kind == "batch":
        t = _batch_sizes(case, 0)
        return int((3 * t + 3 * t // 20).sum()), int(3 * t.sum()), int((t // 2 + 1).sum()), 3
    n0 = 6 * (case["tiles"] * case["quads"]) ** 2
    return n0, n0, (case["tiles"] * case["quads"] + 1) ** 2, 3


def work(case):
    if case["kind"] == "gather":
        es = 8 if case["double"] else 4
        row = es * case["channels"]
        # forward: map, gathered rows in and out; backward: map, rows in, every gradient row out
        return {"bytes": case["new"] * (3 * row + 8) + case["old"] * row, "flops": case["new"] * case["channels"]}
    n, m, u, k = _sizes(case)
    kept = case.get("keep", 1.0)
    # records and entries in; output records, both maps and remapped entries out
    return {"bytes": n * 4 * k + 4 * m + u * 4 * k + 4 * u + 4 * n + int(4 * m * kept) + (m // 3 if kept < 1 else 0),
            "flops": 0}


# ------------------------------------------------------------------- exact


def _exact_mesh(vtx, idx, mesh=None):
    """out_vtx, out_idx, old2new, new2old, U of one mesh by stable sorts of
    the record words (unsigned, first word most significant); `mesh`: the
    vertices' mesh ids, which then come first. Ids are not mesh-local."""
    n = vtx.shape[0]
    words = vtx.contiguous().view(torch.int32).to(torch.int64) & 0xFFFFFFFF
    keys = [words[:, w] for w in range(words.shape[1])]
    if mesh is not None:
        keys.insert(0, mesh)
    order = torch.arange(n, device="cuda")
    for key in reversed(keys):
        order = order[torch.sort(key[order], stable=True).indices]
    head = torch.zeros(n, dtype=torch.bool, device="cuda")
    head[0] = True
    for key in keys:
        s = key[order]
        head[1:] |= s[1:] != s[:-1]
    group = torch.empty(n, dtype=torch.int64, device="cuda")
    group[order] = head.to(torch.int64).cumsum(0) - 1
    used = torch.zeros(int(head.sum()), dtype=torch.bool, device="cuda")
    used[group[idx.reshape(-1).to(torch.int64)]] = True
    new_of = torch.where(used, used.to(torch.int64).cumsum(0) - 1, torch.full_like(used, -1, dtype=torch.int64))
    old2new = new_of[group]
    new2old = order[head][used]
    out_idx = old2new[idx.to(torch.int64)]
    return vtx[new2old], out_idx, old2new, new2old


def _padded(t, n):
    out = torch.zeros((n, *t.shape[1:]), dtype=t.dtype, device=t.device)
    out[: t.shape[0]] = t
    return out


def exact(case, seed):
    s = _inputs(case, seed)
    kind = case["kind"]
    if kind == "gather":
        a, m = s["attrs"].to(torch.float64), s["new2old"].to(torch.int64)
        return {"out": a[m], "grad": torch.zeros_like(a).index_add_(0, m, s["grad"].to(torch.float64))}
    vtx, idx = s["vtx"], s["idx"]
    elems = idx.shape[0]
    vo = s.get("vtx_offsets")
    meta = None
    if kind == "extract":
        idx = idx[s["keep"]]
    if kind in ("batch", "merge"):
        b = torch.arange(vo.numel() - 1, device="cuda")
        mesh_v = torch.repeat_interleave(b, vo.diff())
        idx = idx + vo[torch.repeat_interleave(b, s["elem_offsets"].diff())][:, None]
    out_vtx, out_idx, old2new, new2old = _exact_mesh(vtx, idx, mesh_v if kind == "batch" else None)
    u = new2old.numel()
    out = {}
    if kind == "batch":
        mesh_o = mesh_v[new2old]
        off = torch.searchsorted(mesh_o, torch.arange(vo.numel(), device="cuda"))
        mesh_e = torch.repeat_interleave(b, s["elem_offsets"].diff())
        out_idx = out_idx - off[mesh_e][:, None]
        old2new = torch.where(old2new >= 0, old2new - off[mesh_v], old2new)
        new2old = new2old - vo[mesh_o]
        out["offsets"] = off
    else:
        meta = [u, 0] + ([idx.shape[0]] if kind == "extract" else [])
        out["meta"] = torch.tensor(meta, dtype=torch.int64)
    if case["call"] == "launch":
        out_vtx, new2old = _padded(out_vtx, vtx.shape[0]), _padded(new2old, vtx.shape[0])
        out_idx = _padded(out_idx, elems)
    i32 = torch.int32
    return dict(out, vtx=out_vtx, idx=out_idx.to(i32), old2new=old2new.to(i32), new2old=new2old.to(i32))
