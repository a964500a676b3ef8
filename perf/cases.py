"""The work a program has this framework do, as cases that can be timed and checked.

Every case is one of eight kinds of call, over the range of sizes, types and options in use:

  forward     build a periodic box, cells, densities (and gradients): a snapshot's analysis
  batch       the same for many bounded sub-volumes with buffer particles in one build
  decomposed  a box or a survey volume split into tasks with AUTOBORDER buffers
  train       differentiable cell volumes, a density-matching loss and its position gradient
  deposit     exact average density on a regular grid
  sample      nearest-cell sampling of a field on a regular grid
  tensor      tidal tensor or Hessian of a grid field
  structure   every cell's vertices and faces

``listed`` gives the fixed cases, ``draw`` another one of the same ranges.  ``prepare`` makes a
case's inputs on the GPU (and the built context, where a program has one in hand), ``run`` is
one pass, ``work`` its least bytes and flops, and ``exact`` the same outputs in plain FP64
torch, for the sizes where that takes seconds.
"""
import math

import numpy as np
import torch

import paper_1601_06429_amd as vt

DEV = "cuda"
# the spacing of the 2,097,152-particle box of side 100, to which halo radii are scaled
SPACING_2M = 100.0 / 2_097_152 ** (1.0 / 3.0)
BORDER = 1.5      # buffer thickness of a task in mean spacings (the paper's example)
GHOST = 3.0       # buffer of a batched sub-volume in mean spacings


def listed():
    return [
        # the smallest snapshot: latency and launches of build, cells and densities
        dict(name="forward-4k-uniform", kind="forward", n=4096, dist="uniform", dtype="f64", precision="fp64",
             faces=False),
        # a ragged mid-size snapshot on the mixed-precision path
        dict(name="forward-150k-mixed", kind="forward", n=150_001, dist="clustered", dtype="f32", precision="mixed",
             faces=False),
        # the headline snapshot, with facets kept and the density gradient
        dict(name="forward-2m", kind="forward", n=2_097_152, dist="clustered", dtype="f32", precision="fp64",
             faces=True),
        # a node's share of sub-volumes of very different sizes, one launch for all
        dict(name="batch-24-items", kind="batch", n_items=24, n_lo=3_000, n_hi=60_000, dtype="f32"),
        # an elongated bounded survey volume as slabs, buffers chosen and widened by the library
        dict(name="decomposed-survey-262k", kind="decomposed", n=262_144, layout="slab", tasks=8, dtype="f32"),
        # one step of fitting positions to a target density: forward and backward
        dict(name="train-262k", kind="train", n=262_144, dist="clustered", dtype="f32"),
        # a small FP64 box on an odd, non-cubic grid
        dict(name="deposit-5k-odd", kind="deposit", n=5_003, dist="uniform", dtype="f64", nx=41, ny=29, nz=50),
        # the headline grid
        dict(name="deposit-2m-256", kind="deposit", n=2_097_152, dist="clustered", dtype="f32", nx=256, ny=256,
             nz=256),
        # a quick look at a field: one point per voxel, with the ids of the cells
        dict(name="sample-500k-1pt", kind="sample", n=500_000, dist="clustered", dtype="f32", nx=192, ny=192, nz=192,
             sub=1, nearest=True),
        # a smoother look: several points per voxel
        dict(name="sample-100k-27pt", kind="sample", n=100_000, dist="clustered", dtype="f64", nx=80, ny=72, nz=64,
             sub=3, nearest=False),
        # the tidal tensor of the headline grid
        dict(name="tensor-256-tidal", kind="tensor", nx=256, ny=256, nz=256, tensor="tidal"),
        # the full structure for a viewer
        dict(name="structure-400k", kind="structure", n=400_000, dist="clustered", dtype="f32"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["forward", "forward", "batch", "decomposed", "train", "deposit", "deposit", "sample", "sample",
                       "tensor", "structure"])
    dist = rng.choice(["uniform", "clustered", "clustered"])
    dtype = rng.choice(["f32", "f32", "f64"])
    low = 4_096 if dist == "uniform" else 10_000
    if kind == "forward":
        return dict(kind=kind, n=_log_int(rng, low, 1_500_000), dist=dist, dtype=dtype,
                    precision=rng.choice(["fp64", "fp64", "mixed"]), faces=rng.random() < 0.5)
    if kind == "batch":
        hi = _log_int(rng, 6_000, 100_000)
        return dict(kind=kind, n_items=rng.randint(2, 32), n_lo=max(2_000, hi // rng.randint(2, 20)), n_hi=hi,
                    dtype=dtype)
    if kind == "decomposed":
        return dict(kind=kind, n=_log_int(rng, 30_000, 600_000), layout=rng.choice(["slab", "cube"]),
                    tasks=rng.choice([4, 8, 16]), dtype=dtype)
    if kind == "train":
        return dict(kind=kind, n=_log_int(rng, low, 300_000), dist=dist, dtype=dtype)
    if kind == "deposit":
        n = _log_int(rng, low, 1_200_000)
        side = n ** (1.0 / 3.0) * rng.uniform(0.6, 2.2)
        dims = [min(256, max(8, int(side * rng.uniform(0.7, 1.3)))) for _ in range(3)]
        return dict(kind=kind, n=n, dist=dist, dtype=dtype, nx=dims[0], ny=dims[1], nz=dims[2])
    if kind == "sample":
        sub = rng.choice([1, 1, 1, 2, 3])
        side = _log_int(rng, 24, 224) / (1.0, 1.0, 1.6, 2.2)[sub]
        dims = [max(8, int(side * rng.uniform(0.75, 1.15))) for _ in range(3)]
        return dict(kind=kind, n=_log_int(rng, low, 1_000_000), dist=dist, dtype=dtype, nx=dims[0], ny=dims[1],
                    nz=dims[2], sub=sub, nearest=rng.random() < 0.5)
    if kind == "tensor":
        e = [rng.randint(4, 8) for _ in range(3)]
        return dict(kind=kind, nx=2 ** e[0], ny=2 ** e[1], nz=2 ** e[2], tensor=rng.choice(["tidal", "hessian"]))
    return dict(kind=kind, n=_log_int(rng, low, 500_000), dist=dist, dtype=dtype)


# ----------------------------------------------------------------------------- inputs


def _gen(seed, salt=0):
    return torch.Generator(DEV).manual_seed((int(seed) * 1_000_003 + salt * 7919 + 12345) % (1 << 62))


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device=DEV, dtype=torch.float64)


def _halo_points(g, n, n_halo, lo, size, scale):
    """n points in n_halo NFW-like halos (masses log-uniform over two decades, radii 0.5 - 3 times
    `scale`, concentrations 5 - 15, the radius from the enclosed-mass profile by bisection)."""
    mass = 10.0 ** (2.0 * _rand(g, n_halo))
    centre = lo + _rand(g, n_halo, 3) * size
    radius = (0.5 + 2.5 * _rand(g, n_halo)) * scale
    conc = 5.0 + 10.0 * _rand(g, n_halo)
    h = torch.searchsorted((mass.cumsum(0) / mass.sum()).contiguous(), _rand(g, n)).clamp_(max=n_halo - 1)
    c = conc[h]

    def mu(y):
        return torch.log1p(y) - y / (1.0 + y)

    target = _rand(g, n) * mu(c)
    a, b = torch.zeros_like(c), torch.ones_like(c)
    for _ in range(45):
        m = 0.5 * (a + b)
        below = mu(c * m) < target
        a, b = torch.where(below, m, a), torch.where(below, b, m)
    v = torch.randn(n, 3, generator=g, device=DEV, dtype=torch.float64)
    v /= v.norm(dim=1, keepdim=True)
    return centre[h] + (a * radius[h])[:, None] * v


def _no_duplicates(g, p, lo, size):
    """Exact duplicates (and a few points that only share a hash) drawn again, uniformly."""
    bits = torch.int32 if p.dtype == torch.float32 else torch.int64
    for _ in range(20):
        q = p.view(bits).to(torch.int64)
        key = (q[:, 0] * 0x1F35_79B1_4D2F_9A6B) ^ (q[:, 1] * 0x2545_F491_4F6C_DD1D) ^ (q[:, 2] * 0x1B87_3593_CC9E_2D51)
        s, order = key.sort(stable=True)
        dup = order[1:][s[1:] == s[:-1]]
        if dup.numel() == 0:
            return p
        p[dup] = (lo + _rand(g, dup.numel(), 3) * size).to(p.dtype)
    raise RuntimeError("could not remove duplicate points")


def _periodic_points(g, n, length, dist, dtype):
    lo, size = 0.0, float(length)
    if dist == "uniform":
        p = _rand(g, n, 3) * size
    else:
        scale = size / n ** (1.0 / 3.0) / SPACING_2M
        n_in = n // 2
        halos = _halo_points(g, n_in, max(1, round(200 * n / 2_097_152)), lo, size, scale)
        p = torch.cat([_rand(g, n - n_in, 3) * size, halos]).remainder_(size)
        p = p[torch.randperm(n, generator=g, device=DEV)]
    p = p.to(torch.float32 if dtype == "f32" else torch.float64)
    p = torch.where(p >= size, torch.zeros_like(p), p).contiguous()
    return _no_duplicates(g, p, lo, size)


def _bounded_points(g, n, lo, hi, dtype, spacing):
    """The clustered mix in the bounded box [lo, hi): halo points outside it are drawn uniformly."""
    lo = torch.as_tensor(lo, dtype=torch.float64, device=DEV)
    hi = torch.as_tensor(hi, dtype=torch.float64, device=DEV)
    n_in = n // 2
    halos = _halo_points(g, n_in, max(1, round(200 * n / 2_097_152)), lo, hi - lo, spacing / SPACING_2M)
    p = torch.cat([lo + _rand(g, n - n_in, 3) * (hi - lo), halos])
    t = torch.float32 if dtype == "f32" else torch.float64
    p = p.to(t)
    fresh = (lo + _rand(g, n, 3) * (hi - lo)).to(t)
    inside = ((p.double() > lo) & (p.double() < hi)).all(1, keepdim=True)
    p = torch.where(inside, p, fresh)
    p = torch.minimum(torch.maximum(p, lo.to(t)), torch.nextafter(hi.to(t), lo.to(t)))
    p = p[torch.randperm(n, generator=g, device=DEV)].contiguous()
    return _no_duplicates(g, p, lo, hi - lo)


def _length(case):
    """The box: side 100 for the large FP32 snapshots, the unit cube otherwise."""
    return 100.0 if case["n"] > 100_000 and case["dtype"] == "f32" and case["kind"] != "train" else 1.0


def _masses(g, n):
    return (0.5 + _rand(g, n)).float()


def _batch(case, seed):
    """The items of a batch (sizes log-spaced over the case's range, side ratios up to 2): positions,
    int32 global ids and the item list.  Each item is one clustered field over its buffered box;
    owned and buffer particles are trimmed (or filled uniformly) to the mean's counts."""
    g = _gen(seed)
    r = np.random.default_rng(case["n_items"])
    t = torch.float32 if case["dtype"] == "f32" else torch.float64
    parts, items, off = [], [], 0
    for k in range(case["n_items"]):
        n = int(_item_size(case, k))
        ratio = np.exp(r.uniform(-math.log(2.0), math.log(2.0), 3))
        side = ratio * (n * SPACING_2M ** 3 / np.prod(ratio)) ** (1.0 / 3.0)
        w = GHOST * SPACING_2M
        blo, bhi = -w * np.ones(3), side + w
        m = int(np.prod(bhi - blo) / SPACING_2M ** 3)
        p = _bounded_points(g, m, blo, bhi, case["dtype"], SPACING_2M)
        fill = (torch.as_tensor(blo, device=DEV) + _rand(g, 4 * m, 3) * torch.as_tensor(bhi - blo, device=DEV)).to(t)
        p = torch.cat([p, fill])
        own = ((p.double() >= 0) & (p.double() < torch.as_tensor(side, device=DEV))).all(1)
        n_ghost = m - n
        p = torch.cat([p[own][:n], p[~own][:n_ghost]])
        parts.append(p)
        items.append(dict(offset=off, n_owned=n, n_ghost=n_ghost, periodic=False, lo=blo, hi=bhi))
        off += n + n_ghost
    ids = torch.randperm(off, generator=g, device=DEV).to(torch.int32)
    return torch.cat(parts).contiguous(), ids, items


def _item_size(case, k):
    return case["n_lo"] * (case["n_hi"] / case["n_lo"]) ** (k / max(1, case["n_items"] - 1))


def _built(case, seed, faces):
    """A snapshot that is already tessellated: (context, positions, masses)."""
    g = _gen(seed)
    L = _length(case)
    pos = _periodic_points(g, case["n"], L, case["dist"], case["dtype"])
    ctx = vt.Context().vt_build(pos, vt.whole_box(case["n"], 0.0, L), want_faces=faces)
    return ctx, pos, _masses(g, case["n"])


def _target(x, phase, mean):
    """A smooth periodic target density on the unit box."""
    s = torch.sin(2.0 * math.pi * x / torch.tensor([1.0, 0.5, 1.0 / 3.0], device=x.device, dtype=x.dtype) + phase)
    return mean * (1.0 + 0.5 * s.prod(dim=1))


def _tensor_field(case, seed):
    """A positive field with structure on many scales (a density contrast's shape)."""
    g = _gen(seed)
    shape = (case["nx"], case["ny"], case["nz"])
    f = torch.randn(*shape, generator=g, device=DEV, dtype=torch.float64)
    for d in range(3):
        f = f + torch.roll(f, 1, d) + 0.5 * torch.roll(f, 3, d)
    return torch.exp(0.35 * f).contiguous()


def _cell_arrays(n):
    """A program's own arrays for the cells of n particles, with room for 18 neighbours each."""
    return dict(volume=torch.empty(n, dtype=torch.float64, device=DEV),
                nbr_off=torch.empty(n + 1, dtype=torch.int64, device=DEV),
                nbr_ids=torch.full((18 * n,), -1, dtype=torch.int32, device=DEV),
                status=torch.empty(n, dtype=torch.uint8, device=DEV),
                rho=torch.empty(n, dtype=torch.float64, device=DEV))


def _structure_arrays(n):
    """A viewer's own arrays: 32 vertices, 18 faces and 96 loop entries per cell."""
    return dict(vert_off=torch.empty(n + 1, dtype=torch.int64, device=DEV),
                verts=torch.zeros((32 * n, 3), dtype=torch.float64, device=DEV),
                face_off=torch.empty(n + 1, dtype=torch.int64, device=DEV),
                face_nbr=torch.zeros(18 * n, dtype=torch.int32, device=DEV),
                loop_off=torch.zeros(18 * n + 1, dtype=torch.int64, device=DEV),
                loop_vert=torch.zeros(96 * n, dtype=torch.int32, device=DEV))


def prepare(case, seed):
    kind = case["kind"]
    s = dict(case=case)
    if kind in ("forward", "decomposed"):
        s["out"] = _cell_arrays(case["n"])
    elif kind == "batch":
        s["out"] = _cell_arrays(sum(int(_item_size(case, k)) for k in range(case["n_items"])))
    elif kind == "structure":
        s["out"] = _structure_arrays(case["n"])
    if kind == "forward":
        g = _gen(seed)
        L = _length(case)
        s["pos"] = _periodic_points(g, case["n"], L, case["dist"], case["dtype"])
        s["mass"] = _masses(g, case["n"])
        s["items"] = vt.whole_box(case["n"], 0.0, L)
        s["ctx"] = vt.Context()
        s["precision"] = vt.PREC_MIXED if case["precision"] == "mixed" else vt.PREC_FP64
    elif kind == "batch":
        s["pos"], s["ids"], s["items"] = _batch(case, seed)
        s["mass"] = _masses(_gen(seed, 1), s["pos"].shape[0])
        s["ctx"] = vt.Context()
    elif kind == "decomposed":
        g = _gen(seed)
        n = case["n"]
        if case["layout"] == "slab":
            s["lo"], s["hi"], s["nt"], s["periodic"] = np.zeros(3), np.array([10.0, 1.0, 1.0]), (case["tasks"], 1, 1), False
            s["pos"] = _bounded_points(g, n, s["lo"], s["hi"], case["dtype"], (10.0 / n) ** (1.0 / 3.0))
        else:
            s["lo"], s["hi"], s["nt"], s["periodic"] = np.zeros(3), np.ones(3), vt.task_grid(case["tasks"], "a"), True
            s["pos"] = _periodic_points(g, n, 1.0, "clustered", case["dtype"])
        s["mass"] = _masses(g, n)
        s["ctx"] = vt.Context()
    elif kind == "train":
        g = _gen(seed)
        s["pos"] = _periodic_points(g, case["n"], 1.0, case["dist"], case["dtype"])
        s["phase"] = 2.0 * math.pi * _rand(g, 3)
    elif kind == "deposit":
        s["ctx"], s["pos"], s["mass"] = _built(case, seed, False)
        s["rho"] = s["ctx"].vt_density(s["mass"])
    elif kind == "sample":
        s["ctx"], s["pos"], s["mass"] = _built(case, seed, False)
        s["rho"] = s["ctx"].vt_density(s["mass"])
    elif kind == "tensor":
        pos = _periodic_points(_gen(seed, 2), 4096, 100.0, "uniform", "f32")
        s["ctx"] = vt.Context().vt_build(pos, vt.whole_box(4096, 0.0, 100.0))
        s["pos"] = pos
        s["grid"] = _tensor_field(case, seed)
    else:
        s["ctx"], s["pos"], s["mass"] = _built(case, seed, True)
    return s


# ----------------------------------------------------------------------------- one pass


def _cells(ctx, out, mass):
    ctx.vt_cells_into(out["volume"], out["nbr_off"], out["nbr_ids"], out["status"])
    ctx.vt_density(mass, out=out["rho"])
    return out


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "forward":
        ctx = s["ctx"].vt_build(s["pos"], s["items"], precision=s["precision"], want_faces=case["faces"])
        out = _cells(ctx, s["out"], s["mass"])
        return dict(out, grad=ctx.vt_gradient(out["rho"])) if case["faces"] else out
    if kind == "batch":
        ctx = s["ctx"].vt_build(s["pos"], s["items"], global_id=s["ids"])
        return _cells(ctx, s["out"], s["mass"])
    if kind == "decomposed":
        thick, _ = s["ctx"].vt_decomposed_build(s["pos"], s["lo"], s["hi"], s["nt"], border_factor=BORDER,
                                                periodic=s["periodic"])
        return dict(_cells(s["ctx"], s["out"], s["mass"]), thick=thick)
    if kind == "train":
        pos = s["pos"].detach().requires_grad_(True)
        vol = vt.voronoi_volume(pos, 0.0, 1.0)
        loss = _train_loss(vol, pos, s["phase"])
        (grad,) = torch.autograd.grad(loss, pos)
        return dict(volume=vol.detach(), loss=loss.detach(), grad=grad)
    if kind == "deposit":
        return s["ctx"].vt_grid_deposit(s["rho"], (case["nx"], case["ny"], case["nz"]))
    if kind == "sample":
        return s["ctx"].vt_grid_sample(s["rho"], (case["nx"], case["ny"], case["nz"]), sub=case["sub"],
                                       nearest=case["nearest"])
    if kind == "tensor":
        return s["ctx"].vt_grid_tensor(s["grid"], vt.TENSOR_TIDAL if case["tensor"] == "tidal" else vt.TENSOR_HESSIAN)
    st, out = s["ctx"].vt_structure(), s["out"]
    for name in out:
        v = getattr(st, name)
        out[name][: v.shape[0]].copy_(v)
    return out


def _train_loss(vol, pos, phase):
    rho_t = _target(pos.double(), phase, float(pos.shape[0]))
    return ((torch.log(1.0 / vol) - torch.log(rho_t)) ** 2).mean()


# ----------------------------------------------------------------------------- least work


def work(case):
    """Inputs read once, outputs written once; flops of a cell by the repository's cost model
    (6 per plane within the security radius and vertex, 60 per vertex), a quarter of the mean
    cell's planes being indispensable ones."""
    kind = case["kind"]
    pb = 12 if case.get("dtype") == "f32" else 24
    cell_flops = 6.0 * 30 * 27 + 60.0 * 27
    cell_out = 8 + 8 + 15.5 * 4 + 1 + 8
    if kind == "tensor":
        pts = case["nx"] * case["ny"] * case["nz"]
        return dict(bytes=56.0 * pts, flops=7 * 2.5 * pts * math.log2(pts))
    if kind == "batch":
        n = sum(_item_size(case, k) for k in range(case["n_items"]))
        return dict(bytes=n * (pb + 4 + 4 + cell_out), flops=n * cell_flops)
    n = case["n"]
    if kind == "forward":
        return dict(bytes=n * (pb + 4 + cell_out + (24 if case["faces"] else 0)), flops=n * cell_flops)
    if kind == "decomposed":
        return dict(bytes=n * (pb + 4 + cell_out), flops=n * cell_flops)
    if kind == "train":
        return dict(bytes=n * (pb + 8 + pb), flops=n * (cell_flops + 15.5 * 40))
    if kind == "deposit":
        pts = case["nx"] * case["ny"] * case["nz"]
        # per cell: its faces against the grid columns and planes they meet, about 100 flops each
        return dict(bytes=n * (pb + 8 + 15.5 * 4) + 8.0 * pts, flops=100.0 * (15.5 * n + 20.0 * min(pts, 3 * n)))
    if kind == "sample":
        pts = case["nx"] * case["ny"] * case["nz"]
        return dict(bytes=n * (pb + 8) + pts * (12.0 if case["nearest"] else 8.0),
                    flops=8.0 * 16 * pts * case["sub"] ** 3)
    return dict(bytes=n * (pb + 16 + 27 * 24 + 15.5 * 12 + 81 * 4), flops=n * 27 * 60.0)


# ----------------------------------------------------------------------------- the same in FP64
#
# A cell is the intersection of half-spaces u.y <= h.  In the plane of each face k, every other
# plane l gives a line; the line's part inside all other planes m is the edge (k, l).  With f the
# foot of the origin on plane k and b the distance of the line from f, the face's area is the sum
# of b len / 2 over its edges and the volume the sum of h A / 3, origin inside or not.


def _polytopes(u, h, keep_last=0):
    """Areas, centroids and edge end points of B polytopes given K unit normals and distances each."""
    B, K, _ = u.shape
    ref = torch.where((u[..., :1].abs() < 0.6), torch.tensor([1.0, 0, 0], device=u.device, dtype=u.dtype),
                      torch.tensor([0, 1.0, 0], device=u.device, dtype=u.dtype))
    e1 = torch.linalg.cross(u, ref)
    e1 = e1 / e1.norm(dim=2, keepdim=True)
    e2 = torch.linalg.cross(u, e1)
    dots = (u[:, :, None] * u[:, None]).sum(3)               # u_k . u_l
    ax = (e1[:, :, None] * u[:, None]).sum(3)                # line l in the plane of k: a . s <= b
    ay = (e2[:, :, None] * u[:, None]).sum(3)
    an = torch.sqrt(ax * ax + ay * ay)
    ok = an > 1e-9
    an = torch.where(ok, an, torch.ones_like(an))
    b = (h[:, None, :] - dots * h[:, :, None]) / an
    ax, ay = ax / an, ay / an
    # parallel planes: the one further out bounds nothing, the nearer one everything
    hidden = (~ok & (dots > 0) & ((h[:, None, :] < h[:, :, None]))).any(2)
    px, py = b * ax, b * ay                                  # nearest point of line l to the foot
    num = b[:, :, None, :] - (px[..., None] * ax[:, :, None, :] + py[..., None] * ay[:, :, None, :])
    den = -ay[..., None] * ax[:, :, None, :] + ax[..., None] * ay[:, :, None, :]
    use = ok[:, :, None, :].expand_as(num) & ~torch.eye(K, dtype=torch.bool, device=u.device)
    flat = den.abs() < 1e-13
    t = num / torch.where(flat, torch.ones_like(den), den)
    inf = torch.tensor(math.inf, device=u.device, dtype=u.dtype)
    hi = torch.where(use & ~flat & (den > 0), t, inf).amin(3)
    lo = torch.where(use & ~flat & (den < 0), t, -inf).amax(3)
    out = (use & flat & (num < 0)).any(3)
    live = ok & ~out & (hi > lo) & ~hidden[:, :, None] & torch.isfinite(hi) & torch.isfinite(lo)
    ln = torch.where(live, hi - lo, torch.zeros_like(hi))
    tri = 0.5 * b * ln
    area = tri.sum(2)
    mid = torch.where(live, 0.5 * (hi + lo), torch.zeros_like(hi))
    safe = torch.where(area.abs() > 0, area, torch.ones_like(area))
    cx = (tri * (2.0 / 3.0) * (px - ay * mid)).sum(2) / safe
    cy = (tri * (2.0 / 3.0) * (py + ax * mid)).sum(2) / safe
    foot = h[..., None] * u
    cen = foot + cx[..., None] * e1 + cy[..., None] * e2
    vol = (h * area).sum(1) / 3.0
    ends = None
    if keep_last:
        ends = []
        for w in (lo, hi):
            w = torch.where(live, w, torch.zeros_like(w))
            ends.append((foot[:, :, None] + (px - ay * w)[..., None] * e1[:, :, None]
                         + (py + ax * w)[..., None] * e2[:, :, None]))
        ends = (torch.cat(ends, 2).flatten(1, 2), torch.cat([live, live], 2).flatten(1))
    return area, cen, vol, ends


def _box_planes(x, lo, hi):
    """The six walls of [lo, hi] around the seeds x: unit normals and distances."""
    eye = torch.eye(3, device=DEV, dtype=torch.float64)
    u = torch.stack([-eye[0], eye[0], -eye[1], eye[1], -eye[2], eye[2]])
    h = torch.stack([x[:, 0] - lo[0], hi[0] - x[:, 0], x[:, 1] - lo[1], hi[1] - x[:, 1], x[:, 2] - lo[2],
                     hi[2] - x[:, 2]], 1)
    return u[None].expand(x.shape[0], 6, 3), h


def _cells64(x, lo, hi, periodic, rows=None):
    """Per cell: face neighbours (index, -1 where none), areas, centroids (relative), volume.  Starts
    from the 40 nearest particles and adds, until no vertex has a particle nearer than the seed, the
    particles nearest to the vertices.  None if a cell will not settle."""
    n = x.shape[0]
    L = hi - lo
    rows = torch.arange(n, device=DEV) if rows is None else rows
    K0, F = 40, 72
    nbr = torch.full((rows.numel(), F), -1, device=DEV, dtype=torch.int64)
    area = torch.zeros(rows.numel(), F, device=DEV, dtype=torch.float64)
    cen = torch.zeros(rows.numel(), F, 3, device=DEV, dtype=torch.float64)
    vol = torch.zeros(rows.numel(), device=DEV, dtype=torch.float64)
    chunk = max(1, min(128, int(3e8 / n)))

    def separations(r):
        d = x[None] - x[r][:, None]
        return d - L * torch.round(d / L) if periodic else d

    for c0 in range(0, rows.numel(), chunk):
        at = torch.arange(c0, min(c0 + chunk, rows.numel()), device=DEV)
        idx = None
        for step in range(60):
            r = rows[at]
            d = separations(r)
            d2 = (d * d).sum(2)
            half = 0.5 * d2
            if idx is None:
                idx = d2.scatter(1, r[:, None], math.inf).topk(K0, largest=False).indices
            D = torch.gather(d, 1, idx.clamp(min=0)[..., None].expand(-1, -1, 3))
            dist = D.norm(dim=2)
            none = idx < 0
            u = D / torch.where(none, torch.ones_like(dist), dist)[..., None]
            h = torch.where(none, torch.full_like(dist, 1e3 * float(L.max())), 0.5 * dist)
            if periodic:
                wu, wh = _box_planes(torch.zeros_like(x[r]), -0.5 * L, 0.5 * L)
            else:
                wu, wh = _box_planes(x[r], lo, hi)
            sub = max(1, int(4e8 / (u.shape[1] + 6) ** 3 / 8))
            parts = [_polytopes(torch.cat([u[i:i + sub], wu[i:i + sub]], 1), torch.cat([h[i:i + sub], wh[i:i + sub]], 1), 1)
                     for i in range(0, at.numel(), sub)]
            a = torch.cat([p[0] for p in parts])
            cc = torch.cat([p[1] for p in parts])
            v = torch.cat([p[2] for p in parts])
            # the nearest particle to each vertex: nearer than the seed means the cell is not final
            worst = torch.full((at.numel(), n), -math.inf, device=DEV, dtype=torch.float64)
            q0 = 0
            for p in parts:
                pts, live = p[3]
                m = int(live.sum(1).max())
                sel = live.to(torch.int8).topk(m, dim=1).indices
                pv = torch.gather(pts, 1, sel[..., None].expand(-1, -1, 3))
                pv = torch.where(torch.gather(live, 1, sel)[..., None], pv, torch.zeros_like(pv))
                for j in range(0, m, 24):
                    w = torch.matmul(pv[:, j:j + 24], d[q0:q0 + pv.shape[0]].transpose(1, 2).contiguous())
                    w = w - half[q0:q0 + pv.shape[0], None]
                    worst[q0:q0 + pv.shape[0]] = torch.maximum(worst[q0:q0 + pv.shape[0]], w.amax(1))
                q0 += pv.shape[0]
            worst.scatter_(1, r[:, None], -math.inf)
            worst.scatter_(1, torch.where(none, r[:, None], idx), -math.inf)
            size2 = v.clamp(min=0) ** (2.0 / 3.0)
            bad, who = worst.topk(32, dim=1)
            more = bad > 1e-12 * size2[:, None]
            final = ~more.any(1)
            faces = a[:, :-6] > 1e-12 * size2[:, None]
            if bool((faces.sum(1) > F).any()):
                return None
            order = torch.where(faces & ~none, a[:, :-6], torch.zeros_like(a[:, :-6])).topk(min(F, a.shape[1] - 6), dim=1)
            keep = order.values > 0
            face_idx = torch.where(keep, torch.gather(idx, 1, order.indices), torch.full_like(order.indices, -1))
            k = order.indices.shape[1]
            done = at[final]
            nbr[done, :k] = face_idx[final]
            area[done, :k] = order.values[final]
            cen[done, :k] = torch.gather(cc, 1, order.indices[..., None].expand(-1, -1, 3))[final]
            vol[done] = v[final]
            if bool(final.all()):
                break
            idx = torch.cat([face_idx, torch.where(more, who, torch.full_like(who, -1))], 1)[~final]
            idx = idx[:, (idx >= 0).any(0)]
            at = at[~final]
        else:
            return None
    return nbr, area, cen, vol


def _density_gradient64(x, L, nbr, rho):
    d = x[nbr.clamp(min=0)] - x[:, None]
    d = torch.where((nbr >= 0)[..., None], d - L * torch.round(d / L), torch.zeros_like(d))
    dr = rho[nbr.clamp(min=0)] - rho[:, None]
    G = (d[..., :, None] * d[..., None, :]).sum(1)
    return torch.linalg.solve(G, (dr[..., None] * d).sum(1))


def _plain(s):
    return dict(volume=s, nbr_off=None, nbr_ids=None, status=None)


def _exact_tensor(case, seed):
    f = _tensor_field(case, seed)
    shape = f.shape
    F = torch.fft.fftn(f / f.mean() if case["tensor"] == "tidal" else f)
    m = [torch.fft.fftfreq(k, 1.0 / k, device=DEV, dtype=torch.float64).round() for k in shape]
    k = [2.0 * math.pi * m[a].reshape([-1 if b == a else 1 for b in range(3)]) / 100.0 for a in range(3)]
    k2 = k[0] ** 2 + k[1] ** 2 + k[2] ** 2
    nyq = [(m[a] == -(shape[a] // 2)).reshape([-1 if b == a else 1 for b in range(3)]) for a in range(3)]
    out = []
    for i, j in ((0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2)):
        w = k[i] * k[j] + 0.0 * k2
        w = w / torch.where(k2 > 0, k2, torch.ones_like(k2)) if case["tensor"] == "tidal" else -w
        if i != j:
            w = torch.where(nyq[i] | nyq[j], torch.zeros_like(w), w)
        out.append(torch.fft.ifftn(w * F).real)
    return torch.stack(out)


def _exact_sample(case, pos, rho):
    x = pos.double()
    L = _length(case)
    dims = (case["nx"], case["ny"], case["nz"])
    sub = case["sub"]
    ax = [((torch.arange(d * sub, device=DEV, dtype=torch.float64) // sub)
           + ((torch.arange(d * sub, device=DEV, dtype=torch.float64) % sub) + 0.5) / sub) * (L / d) for d in dims]
    q = torch.stack(torch.meshgrid(*ax, indexing="ij"), -1).reshape(-1, 3)
    near = torch.empty(q.shape[0], dtype=torch.int64, device=DEV)
    step = max(1, int(2e8 / x.shape[0]))
    for i in range(0, q.shape[0], step):
        d2 = 0.0
        for a in range(3):
            e = q[i:i + step, a, None] - x[None, :, a]
            d2 = d2 + (e - L * torch.round(e / L)) ** 2
        near[i:i + step] = d2.argmin(1)
    v = rho[near].reshape(dims[0], sub, dims[1], sub, dims[2], sub).mean(dim=(1, 3, 5))
    return (v, None) if case["nearest"] else v


def _exact_deposit(case, pos, mass):
    x = pos.double()
    L = _length(case)
    box = torch.full((3,), L, device=DEV, dtype=torch.float64)
    got = _cells64(x, torch.zeros_like(box), box, True)
    if got is None:
        return None
    nbr, _, _, vol = got
    dims = torch.tensor([case["nx"], case["ny"], case["nz"]], device=DEV)
    hvox = box / dims
    d = x[nbr.clamp(min=0)] - x[:, None]
    d = d - L * torch.round(d / L)
    F = int((nbr >= 0).sum(1).max())
    d, none = d[:, :F], (nbr < 0)[:, :F]
    dist = torch.where(none, torch.ones_like(d[..., 0]), d.norm(dim=2))
    u = d / dist[..., None]
    u = torch.where(none[..., None], torch.tensor([1.0, 0.0, 0.0], device=DEV, dtype=torch.float64), u)
    h = torch.where(none, torch.full_like(dist, 1e3 * L), 0.5 * dist)
    wu, wh = _box_planes(torch.zeros_like(x), -0.5 * box, 0.5 * box)
    ext = torch.zeros(x.shape[0], 3, 2, device=DEV, dtype=torch.float64)
    for i in range(0, x.shape[0], 256):
        pts, live = _polytopes(torch.cat([u[i:i + 256], wu[i:i + 256]], 1), torch.cat([h[i:i + 256], wh[i:i + 256]], 1), 1)[3]
        ext[i:i + 256, :, 0] = torch.where(live[..., None], pts, torch.full_like(pts, math.inf)).amin(1)
        ext[i:i + 256, :, 1] = torch.where(live[..., None], pts, torch.full_like(pts, -math.inf)).amax(1)
    i0 = torch.floor((x + ext[..., 0]) / hvox).long()
    cnt = torch.floor((x + ext[..., 1]) / hvox).long() - i0 + 1
    tot = cnt.prod(1)
    if int(tot.sum()) > 1_500_000:
        return None
    cell = torch.repeat_interleave(torch.arange(x.shape[0], device=DEV), tot)
    k = torch.arange(cell.numel(), device=DEV) - (tot.cumsum(0) - tot)[cell]
    cz = cnt[cell]
    vox = i0[cell] + torch.stack([k // (cz[:, 1] * cz[:, 2]), (k // cz[:, 2]) % cz[:, 1], k % cz[:, 2]], 1)
    rho = mass.double() / vol
    grid = torch.zeros(tuple(dims.tolist()), device=DEV, dtype=torch.float64).reshape(-1)
    step = max(1, int(1.2e8 / (F + 6) ** 3))
    for i in range(0, cell.numel(), step):
        c, w = cell[i:i + step], vox[i:i + step]
        # about the voxel's own centre, which keeps the sums of the size of the voxel
        o = (w + 0.5) * hvox - x[c]
        hh = h[c] - (u[c] * o[:, None]).sum(2)
        bu, bh = _box_planes(torch.zeros_like(o), -0.5 * hvox, 0.5 * hvox)
        v = _polytopes(torch.cat([u[c], bu], 1), torch.cat([hh, bh], 1))[2]
        m = w.remainder(dims)
        grid.index_add_(0, (m[:, 0] * dims[1] + m[:, 1]) * dims[2] + m[:, 2], rho[c] * v.clamp(min=0) / hvox.prod())
    return grid.reshape(tuple(dims.tolist()))


def exact(case, seed):
    kind = case["kind"]
    if kind == "tensor":
        return _exact_tensor(case, seed)
    if kind in ("structure", "batch"):
        return None
    n = case["n"]
    if kind == "sample":
        if n * case["nx"] * case["ny"] * case["nz"] * case["sub"] ** 3 > 4e11:
            return None
        ctx_free = _gen(seed)
        pos = _periodic_points(ctx_free, n, _length(case), case["dist"], case["dtype"])
        mass = _masses(ctx_free, n)
        box = torch.full((3,), _length(case), device=DEV, dtype=torch.float64)
        got = _cells64(pos.double(), torch.zeros_like(box), box, True) if n <= 25_000 else None
        return None if got is None else _exact_sample(case, pos, mass.double() / got[3])
    if n > 25_000:
        return None
    g = _gen(seed)
    if kind == "deposit":
        pos = _periodic_points(g, n, _length(case), case["dist"], case["dtype"])
        return _exact_deposit(case, pos, _masses(g, n)) if n <= 12_000 else None
    if kind == "forward":
        pos = _periodic_points(g, n, _length(case), case["dist"], case["dtype"])
        mass = _masses(g, n)
        box = torch.full((3,), _length(case), device=DEV, dtype=torch.float64)
        got = _cells64(pos.double(), torch.zeros_like(box), box, True)
        if got is None:
            return None
        rho = mass.double() / got[3]
        out = _plain(got[3])
        out["rho"] = rho
        if case["faces"]:
            out["grad"] = _density_gradient64(pos.double(), box, got[0], rho)
        return out
    if kind == "train":
        pos = _periodic_points(g, n, 1.0, case["dist"], case["dtype"])
        phase = 2.0 * math.pi * _rand(g, 3)
        box = torch.ones(3, device=DEV, dtype=torch.float64)
        got = _cells64(pos.double(), torch.zeros_like(box), box, True)
        if got is None:
            return None
        nbr, area, cen, vol = got
        v = vol.clone().requires_grad_(True)
        p = pos.double().clone().requires_grad_(True)
        loss = _train_loss(v, p, phase)
        gv, gp = torch.autograd.grad(loss, (v, p))
        d = p.detach()[nbr.clamp(min=0)] - p.detach()[:, None]
        dist = torch.where(nbr >= 0, (d - torch.round(d)).norm(dim=2), torch.ones_like(area))
        w = (gv[:, None] - gv[nbr.clamp(min=0)]) * area / dist
        return dict(volume=vol, loss=loss.detach(), grad=gp + (w[..., None] * cen).sum(1))
    return None
