"""The work that a user has this framework do, as timed cases.

One pass of a case renders the frames of `cameras` views of a resident mesh through the library's public entry
points, each view different from the one before (a camera that moves, or a stream of requests), and returns the
moment images and the colour images.  `path` says how a program asks for its frames:

  frame   all subdomains on this GPU: stage one sums them itself, stage two walks the rays again and finalises
  server  Server.render: requests of one size, small ones walked by (tile, subdomain) pairs
  ranks   every subdomain apart, as ranks that exchange images would: moments per subdomain, their sum, one
          additive colour image per subdomain, their sum
  tiles   as `ranks`, but the moments as the non-empty tiles that ranks would send
  kept    as `frame`, stage one keeping its pieces for stage two
  f16     as `frame`, the moment image handed on in its packed FP16 form
  graph   as `frame`, each view captured once in a HIP graph and replayed

Sizes are those of the repository's own workloads (16^3 to 128^3 cubes of six tets, 4 to 72 subdomains, images of
128^2 to 2560^2 pixels, 4, 6 or 8 moments, orthographic and perspective) with odd ones between.  A graded mesh has
cells eight times finer in the middle than at its ends and subdomains whose tet counts differ by up to a factor of
12, like the adaptive workload.
"""
import math

import numpy as np
import torch

import paper_2501_12581_amd as apc

KAPPA, CAP, ALPHA, ETA, TABLE = 4.0, 10.0, 5e-5, 0.3, 256


def listed():
    def case(name, path, n, subs, w, h, m, cameras=2, ortho=False, graded=False):
        return dict(name=name, path=path, n=n, subs=subs, w=w, h=h, m=m, cameras=cameras, ortho=ortho, graded=graded)

    return [
        # the smallest workload: a preview of a small volume, where launches and round trips count
        case("tiny_frame", "frame", 16, 4, 128, 128, 4, ortho=True),
        # render requests as a server meets them: thumbnails, ordinary views, full views
        case("request_256", "server", 64, 72, 256, 256, 8, graded=True),
        case("request_512", "server", 64, 72, 512, 512, 6, graded=True),
        case("request_1024", "server", 64, 72, 1024, 1024, 4, graded=True),
        # an odd window size, neither side a multiple of a tile
        case("ragged_frame", "frame", 48, 16, 643, 427, 8),
        # the ordinary frame of a medium volume
        case("medium_frame", "frame", 64, 16, 1024, 1024, 6),
        # uneven subdomains on cells of very different sizes
        case("graded_frame", "frame", 64, 72, 1024, 1024, 8, graded=True),
        # what the ranks of a distributed run compute: dense images, and non-empty tiles
        case("rank_images", "ranks", 48, 8, 512, 512, 6, cameras=1),
        case("rank_tiles", "tiles", 48, 16, 640, 480, 8, cameras=1),
        # the kept-piece variant and a replayed graph
        case("kept_frame", "kept", 64, 16, 1024, 1024, 8),
        case("graph_frame", "graph", 32, 16, 512, 512, 6),
        # the largest: a volume of 12.6M tets filling a 2560^2 image
        case("large_frame", "frame", 128, 72, 2560, 2560, 8, cameras=1),
    ]


def draw(rng):
    def between(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    path = rng.choice(["frame", "frame", "frame", "server", "server", "tiles", "ranks", "kept", "f16", "graph"])
    n, m = between(12, 96), rng.choice([4, 6, 8])
    side = between(96, 1400)
    if path == "server":
        w = h = side
    else:
        w, h = side, max(33, int(side * rng.uniform(0.5, 1.2)))
    subs = between(2, 72)
    if path == "ranks":  # a dense image per subdomain
        subs, w, h = min(subs, 12), min(w, 700), min(h, 700)
    return dict(path=path, n=n, subs=subs, w=w, h=h, m=m, cameras=rng.choice([1, 2]),
                ortho=path != "server" and rng.random() < 0.25, graded=rng.random() < 0.4)


# ------------------------------------------------------------------------------------------------ inputs

def _device():
    return torch.device("cuda:0" if torch.cuda.is_available() else "cpu")


def _grade(x):
    """A monotone map of [0, 1] onto itself, its slope 1/4 in the middle and 5/2 at the ends."""
    u = 2.0 * x - 1.0
    return 0.5 + 0.5 * u * (0.25 + 0.75 * u * u)


_PATHS = ((0, 1, 2), (1, 2, 0), (2, 0, 1), (1, 0, 2), (0, 2, 1), (2, 1, 0))  # three even, three odd


def _mesh(case, seed):
    """A jittered grid of n^3 cubes, six tets each around the main diagonal, cubes in Morton order, cut into runs
    of cubes as subdomains; a sum of Gaussians as the scalar.  (xyz, scalar, tets, tet_sub) on the device."""
    n, dev = case["n"], _device()
    rng = np.random.default_rng([seed, n])
    g = torch.Generator(device=dev).manual_seed(int(rng.integers(1 << 62)))
    line = torch.arange(n + 1, device=dev)
    k, j, i = torch.meshgrid(line, line, line, indexing="ij")
    idx = torch.stack([i.ravel(), j.ravel(), k.ravel()], dim=1)
    jitter = (torch.rand(idx.shape, generator=g, device=dev, dtype=torch.float64) * 2 - 1) * 0.15
    jitter[(idx == 0) | (idx == n)] = 0.0
    xyz = (idx + jitter) / n
    if case["graded"]:
        xyz = _grade(xyz)
    centres = torch.as_tensor(rng.uniform(0.2, 0.8, size=(12, 3)), device=dev)
    scalar = torch.zeros(len(xyz), device=dev, dtype=torch.float64)
    for c in centres:
        scalar += torch.exp(((xyz - c) ** 2).sum(dim=1) / (-2.0 * 0.15 * 0.15))
    cell = torch.arange(n, device=dev)
    k, j, i = torch.meshgrid(cell, cell, cell, indexing="ij")
    code = torch.zeros(n ** 3, device=dev, dtype=torch.int64)
    for b in range(max(1, (n - 1).bit_length())):
        for axis, v in enumerate((i, j, k)):
            code |= ((v.ravel() >> b) & 1) << (3 * b + axis)
    order = torch.argsort(code)
    base = (i + (n + 1) * (j + (n + 1) * k)).ravel()[order]
    step = (1, n + 1, (n + 1) * (n + 1))
    tets = torch.empty((n ** 3, 6, 4), device=dev, dtype=torch.int32)
    for t, (a, b, _) in enumerate(_PATHS):
        mid = [base + step[a], base + step[a] + step[b]]
        if t >= 3:
            mid.reverse()
        for q, v in enumerate([base] + mid + [base + sum(step)]):
            tets[:, t, q] = v.to(torch.int32)
    subs = case["subs"]
    ratio = 12.0 if case["graded"] else 2.0
    weight = rng.permutation(ratio ** (np.arange(subs) / max(1, subs - 1)))
    cut = np.rint(np.concatenate([[0.0], np.cumsum(weight)]) / weight.sum() * n ** 3).astype(np.int64)
    of_cube = torch.bucketize(torch.arange(n ** 3, device=dev), torch.as_tensor(cut[1:-1], device=dev), right=True)
    return (xyz.to(torch.float32).contiguous(), scalar.to(torch.float32).contiguous(),
            tets.reshape(-1, 4).contiguous(), of_cube.to(torch.int32).repeat_interleave(6).contiguous())


def _cameras(case, seed):
    """Views of the unit cube's centre from seeded points of the sphere of radius 2."""
    rng = np.random.default_rng([seed, 77])
    out = []
    for _ in range(case["cameras"]):
        v = rng.normal(size=3)
        eye = 0.5 + 2.0 * v / np.linalg.norm(v)
        f = (0.5 - eye) / 2.0
        up = np.array([0.0, 0.0, 1.0]) if abs(f[2]) <= 0.99 else np.array([0.0, 1.0, 0.0])
        r = np.cross(f, up)
        r /= np.linalg.norm(r)
        d = np.cross(f, r)
        w, h = case["w"], case["h"]
        if case["ortho"]:  # a window 1.8 wide and high around the axis
            right, down = r * (1.8 / w), d * (1.8 / h)
            eye = eye - 0.9 * r - 0.9 * d
        else:
            half = math.tan(math.radians(45.0) / 2.0)
            right, down = r * (2.0 * half / h), d * (2.0 * half / h)
        out.append(dict(width=w, height=h, projection=0 if case["ortho"] else 1, eye=tuple(eye), dir=tuple(f),
                        right=tuple(right), down=tuple(down)))
    return out


def _table(seed):
    """RGBA transfer function through four seeded control points."""
    rng = np.random.default_rng([seed, 11])
    at, col = np.sort(rng.uniform(0, 1, 4)), rng.uniform(0, 1, (4, 4))
    x = np.arange(TABLE) / (TABLE - 1)
    return np.stack([np.interp(x, at, col[:, c]) for c in range(4)], axis=1).astype(np.float32)


def _bias(m):
    j = np.arange(1, m + 1)
    return np.where(j % 2 == 0, 1.0 / (j + 1.0), 0.0)


def _range(scalar):
    return float(scalar.min()), float(scalar.max())


def _step(case):
    return 0.25 / case["n"]


# ------------------------------------------------------------------------------------------------ passes

class _State:
    pass


def prepare(case, seed):
    dev, s = _device(), _State()
    s.case = case
    arrays = _mesh(case, seed)
    lo, hi = _range(arrays[1])
    m, subs, w, h = case["m"], case["subs"], case["w"], case["h"]
    views = _cameras(case, seed)
    if case["path"] == "server":
        from paper_2501_12581_amd.serve import Server
        s.server = Server(arrays + (subs,), _step(case), [_table(seed)], (lo, hi), slots=1, max_size=w, max_m=m,
                          by_pair=True)
        s.server.warm(eye=views[0]["eye"])
        s.requests = [dict(id=k, arrival=0.0, size=w, eye=v["eye"], m=m, tf=0) for k, v in enumerate(views)]
        return s
    s.ctx = apc.Context(0)
    s.mesh = s.ctx.load_mesh(*arrays, subs)
    s.table = torch.as_tensor(_table(seed), device=dev)
    s.tf = apc.make_tf(s.table, lo, hi, KAPPA, CAP)
    s.mboit = apc.make_mboit(m, ALPHA, _bias(m), ETA)
    s.subs = np.arange(subs, dtype=np.int32)
    s.views = [apc.make_view(v, _step(case)) for v in views]
    s.moments = [torch.zeros((m + 1, h, w), device=dev) for _ in views]
    s.rgba = [torch.zeros((h, w, 4), device=dev) for _ in views]
    if case["path"] == "ranks":
        s.per_sub = torch.zeros((subs, m + 1, h, w), device=dev)
    if case["path"] in ("ranks", "tiles"):
        s.partial = torch.zeros((subs if case["path"] == "ranks" else 2, h, w, 4), device=dev)
    if case["path"] == "tiles":
        pairs = max(s.ctx.moments_pass_tiles(s.mesh, v, s.tf, m, s.subs) for v in s.views)
        s.tiles = torch.zeros((pairs, m + 1, 64), device=dev)
        s.bins = torch.zeros(pairs, dtype=torch.int32, device=dev)
    if case["path"] == "f16":
        s.packed = [torch.zeros((m + 3, h, w), dtype=torch.float16, device=dev) for _ in views]
    if case["path"] == "kept":  # the library grows its piece store to what such a frame needs
        for k in range(2 * len(s.views)):
            _frame(s, k % len(s.views))
        torch.cuda.synchronize()
    if case["path"] == "graph":
        s.graphs = []
        for k, v in enumerate(s.views):
            r = _State()
            r.ctx, r.mesh, r.view, r.tf, r.mboit, r.subs = s.ctx, s.mesh, v, s.tf, s.mboit, s.subs
            r.moments, r.rgba = s.moments[k], s.rgba[k]
            s.graphs.append(apc.FrameGraph(r, global_sum=True))
    return s


def _frame(s, k):
    path, m, view, mom, rgba = s.case["path"], s.case["m"], s.views[k], s.moments[k], s.rgba[k]
    if path == "graph":
        s.graphs[k].launch()
        return [mom, rgba]
    if path == "ranks":
        s.ctx.moments_pass(s.mesh, view, s.tf, m, s.subs, s.per_sub)
        s.ctx.sum_moments(s.per_sub, m, s.subs, mom)
        for q in range(len(s.subs)):
            s.ctx.resolve_pass(s.mesh, view, s.tf, s.mboit, mom, s.subs[q:q + 1], s.partial[q], finalize=False)
        s.ctx.sum_images(s.partial, s.subs, mom, s.mboit, rgba)
        return [s.per_sub, mom, s.partial, rgba]
    if path == "tiles":  # two ranks, each with half of the subdomains
        n = s.ctx.moments_pass_tiles(s.mesh, view, s.tf, m, s.subs, s.tiles, s.bins)
        s.ctx.sum_moment_tiles(s.tiles, s.bins, n, len(s.subs), m, view.height, view.width, mom)
        half = len(s.subs) // 2
        for q, own in enumerate((s.subs[:half], s.subs[half:])):
            s.ctx.resolve_pass(s.mesh, view, s.tf, s.mboit, mom, own, s.partial[q], finalize=False, by_pair=True)
        s.ctx.sum_images(s.partial, None, mom, s.mboit, rgba)
        return [mom, s.partial, rgba]
    s.ctx.moments_pass(s.mesh, view, s.tf, m, s.subs, mom, keep=path == "kept", global_sum=True)
    if path == "f16":
        s.ctx.pack_moments_f16(mom, m, s.packed[k])
        s.ctx.resolve_pass(s.mesh, view, s.tf, s.mboit, s.packed[k], s.subs, rgba)
        return [mom, s.packed[k], rgba]
    s.ctx.resolve_pass(s.mesh, view, s.tf, s.mboit, mom, s.subs, rgba)
    return [mom, rgba]


def run(s):
    if s.case["path"] == "server":  # the image is the slot's buffer: the client's copy of it comes back
        return [[s.server.render(0, req).clone()] for req in s.requests]
    return [_frame(s, k) for k in range(len(s.views))]


def _counts(case):
    """Rays that meet the cube, tets and pieces along them, for a mean view of an even mesh."""
    n, px = case["n"], case["w"] * case["h"]
    seen = 1.5 / (1.8 * 1.8) if case["ortho"] else 1.5 / (4.0 * math.tan(math.radians(22.5))) ** 2 * case["h"] / case["w"]
    rays = px * min(1.0, seen)
    return rays, rays * 2.4 * n, rays * 5.07 * n


def work(case):
    """The mesh read once and the images written once; a tet crossed and a piece evaluated once (a step about 100
    operations, a piece's moments 2 (m + 1), its moment bound about 250 at m = 8, 150 at 6, 60 at 4)."""
    n, px, m = case["n"], case["w"] * case["h"], case["m"]
    rays, steps, pieces = _counts(case)
    size = 16 * (n + 1) ** 3 + 6 * n ** 3 * 32
    image = px * (4 * (m + 1) + 16)
    if case["path"] == "ranks":
        image += px * case["subs"] * (4 * (m + 1) + 16)
    flops = steps * 100 + pieces * (2 * (m + 1) + {4: 60, 6: 150, 8: 250}[m])
    return {"bytes": float(case["cameras"] * (size + image)), "flops": float(case["cameras"] * flops)}


# ------------------------------------------------------------------------------------------------ in 64 bits

def exact(case, seed):
    """The same frames in 64 bits from the method's formulas: every tet clipped against the pixel rays of its
    projected box, chords cut at the lattice, moments added; then per pixel the biased moments' Jacobi matrix,
    and per piece the nodes of the bound by bisection between the zeros of the orthonormal polynomial."""
    _, _, pieces = _counts(case)
    if pieces > 3e9 or not torch.cuda.is_available():
        return None
    xyz, scalar, tets, of = _mesh(case, seed)
    table = torch.as_tensor(_table(seed), device=_device()).double()
    out = []
    for view in _cameras(case, seed):
        whole = pieces <= 4e8
        parts = case["subs"] if case["path"] == "ranks" else 2 if case["path"] == "tiles" else 1
        part = of.long() if case["path"] == "ranks" else (of.long() >= case["subs"] // 2).long() * (parts - 1)
        per, kept = _stage_one(xyz.double(), scalar.double(), tets.long(), part, parts, view, _step(case),
                               case["m"], table, _range(scalar), whole)
        mom = per.sum(dim=0)
        h, w = case["h"], case["w"]
        image = mom.reshape(-1, h, w)
        cols = rgba = None
        if whole:
            cols = _stage_two(mom, kept, parts, table, case["m"])
            a = -torch.expm1(-mom[0])
            total = cols.sum(dim=0)
            rgba = (torch.cat([total[:, :3] * (a / total[:, 3].clamp(min=1e-30))[:, None], a[:, None]], dim=1)
                    * (total[:, 3:] > 1e-30)).reshape(h, w, 4)
            cols = cols.reshape(parts, h, w, 4)
        del kept
        if case["path"] == "server":
            out.append([rgba])
        elif case["path"] == "ranks":
            out.append([per.reshape(parts, -1, h, w), image, cols, rgba])
        elif case["path"] == "tiles":
            out.append([image, cols, rgba])
        elif case["path"] == "f16":
            out.append([image, None, rgba])
        else:
            out.append([image, rgba])
    return out


def _rays(view, pix):
    w, h = view["width"], view["height"]
    a, b = (pix % w).double() + 0.5, (pix // w).double() + 0.5
    eye, d, right, down = (torch.tensor(view[k], device=pix.device, dtype=torch.float64)
                           for k in ("eye", "dir", "right", "down"))
    if view["projection"] == 0:
        return eye + a[:, None] * right + b[:, None] * down, (d / d.norm()).expand(len(pix), 3)
    d = d + (a - 0.5 * w)[:, None] * right + (b - 0.5 * h)[:, None] * down
    return eye.expand(len(pix), 3), d / d.norm(dim=1, keepdim=True)


def _depths(view, xyz):
    lo, hi = xyz.min(dim=0).values, xyz.max(dim=0).values
    off = 0.5 * (lo + hi) - torch.tensor(view["eye"], device=xyz.device, dtype=torch.float64)
    d = torch.tensor(view["dir"], device=xyz.device, dtype=torch.float64)
    dist = float(off.norm() if view["projection"] else off @ (d / d.norm()))
    r = 0.5 * float((hi - lo).norm())
    return dist - r, dist + r


def _stage_one(xyz, scalar, tets, part, parts, view, step, m, table, rng, keep):
    dev, w, h = xyz.device, view["width"], view["height"]
    near, far = _depths(view, xyz)
    eye, d, right, down = (torch.tensor(view[k], device=dev, dtype=torch.float64) for k in ("eye", "dir", "right", "down"))
    inv = torch.linalg.inv(torch.stack([d, right, down], dim=1))
    l, u, v = ((xyz - eye) @ inv.T).unbind(dim=1)
    col = u - 0.5 if view["projection"] == 0 else u / l + 0.5 * w - 0.5
    row = v - 0.5 if view["projection"] == 0 else v / l + 0.5 * h - 0.5
    c0 = torch.ceil(col[tets].min(dim=1).values - 1e-6).clamp(min=0).long()
    c1 = torch.floor(col[tets].max(dim=1).values + 1e-6).clamp(max=w - 1).long()
    r0 = torch.ceil(row[tets].min(dim=1).values - 1e-6).clamp(min=0).long()
    r1 = torch.floor(row[tets].max(dim=1).values + 1e-6).clamp(max=h - 1).long()
    many = (c1 - c0 + 1).clamp(min=0) * (r1 - r0 + 1).clamp(min=0)
    ends = torch.cumsum(many, dim=0)
    total, most = int(ends[-1]), 1 << 24
    mom = torch.zeros((parts * w * h, m + 1), device=dev, dtype=torch.float64)
    kept, first = [], 0
    cuts = torch.searchsorted(ends, torch.arange(most, total + most, most, device=dev), right=True).tolist()
    for last in cuts[:-1] + [len(tets)]:
        t = torch.arange(first, last, device=dev)
        first = last
        t = t[many[t] > 0]
        if not len(t):
            continue
        rep = torch.repeat_interleave(torch.arange(len(t), device=dev), many[t])
        k = torch.arange(len(rep), device=dev) - (torch.cumsum(many[t], dim=0) - many[t])[rep]
        wide = (c1 - c0 + 1)[t][rep]
        pix = (r0[t][rep] + k // wide) * w + c0[t][rep] + k % wide
        o, ray = _rays(view, pix)
        p = xyz[tets[t]]
        t0 = torch.full((len(rep),), -math.inf, device=dev, dtype=torch.float64)
        t1 = torch.full((len(rep),), math.inf, device=dev, dtype=torch.float64)
        sc, grad = scalar[tets[t]], torch.zeros((len(t), 3), device=dev, dtype=torch.float64)
        for apex, f in enumerate(((1, 2, 3), (0, 3, 2), (0, 1, 3), (0, 2, 1))):  # outward, opposite vertex `apex`
            normal = torch.linalg.cross(p[:, f[1]] - p[:, f[0]], p[:, f[2]] - p[:, f[0]])
            height = (normal * (p[:, apex] - p[:, f[0]])).sum(dim=1)
            grad += normal * (sc[:, apex] / height)[:, None]
            den = (normal[rep] * ray).sum(dim=1)
            at = (normal[rep] * (p[:, f[0]][rep] - o)).sum(dim=1) / den
            t0 = torch.where(den < 0, torch.maximum(t0, at), t0)
            t1 = torch.where(den > 0, torch.minimum(t1, at), t1)
        hit = t1 > t0
        rep, pix, o, ray, t0, t1 = rep[hit], pix[hit], o[hit], ray[hit], t0[hit], t1[hit]
        s_at = sc[:, 0][rep] + (grad[rep] * (o - p[:, 0][rep])).sum(dim=1)
        slope = (grad[rep] * ray).sum(dim=1)
        k0 = torch.floor((t0 - near) / step)
        slot = part[t][rep] * (w * h) + pix
        for i in range(int((torch.ceil((t1 - near) / step) - k0).max()) + 1 if len(t0) else 0):
            a, b = torch.maximum(t0, near + (k0 + i) * step), torch.minimum(t1, near + (k0 + i + 1) * step)
            on = b > a
            mid, size = 0.5 * (a + b)[on], (b - a)[on]
            s = s_at[on] + slope[on] * mid
            x = ((s - rng[0]) * ((len(table) - 1) / (rng[1] - rng[0]))).clamp(0, len(table) - 1)
            lo = x.long().clamp(max=len(table) - 2)
            al = table[:, 3][lo] + (table[:, 3][lo + 1] - table[:, 3][lo]) * (x - lo)
            dep = (KAPPA * al * size).clamp(max=CAP)
            z = (2.0 * torch.log(mid / near) / math.log(far / near) - 1.0).clamp(-1, 1)
            power = z[:, None] ** torch.arange(m + 1, device=dev)
            mom.index_add_(0, slot[on], dep[:, None] * power)
            if keep:
                kept.append((slot[on].int(), z, dep, x))
    return mom.reshape(parts, w * h, m + 1).transpose(1, 2).contiguous(), kept


def _stage_two(mom, kept, parts, table, m):
    dev, n, px = mom.device, m // 2, mom.shape[1]
    seen = torch.nonzero(mom[0] > 0).squeeze(1)
    beta = (1 - ALPHA) * mom[:, seen] / mom[0, seen]
    beta[1:] += ALPHA * torch.as_tensor(_bias(m), device=dev)[:, None]
    beta[0] = 1.0
    up = {}  # the upper Cholesky factor of the Hankel matrix beta_(i+j)
    for i in range(n + 1):
        for j in range(i, n + 1):
            v = beta[i + j] - sum(up[k, i] * up[k, j] for k in range(i))
            up[i, j] = torch.sqrt(v) if i == j else v / up[i, i]
    # the Jacobi matrix of the biased moments (diagonal a_k, off-diagonal b_k) from that factor
    b = [up[k, k] / up[k - 1, k - 1] for k in range(1, n + 1)]
    q = [up[k, k + 1] / up[k, k] for k in range(n)]
    a = [q[0]] + [q[k] - q[k - 1] for k in range(1, n)]
    jac = torch.zeros((len(seen), n, n), dtype=torch.float64)
    for k in range(n):
        jac[:, k, k] = a[k].cpu()
        if k + 1 < n:
            jac[:, k, k + 1] = jac[:, k + 1, k] = b[k].cpu()
    zeros, vec = torch.linalg.eigh(jac)
    place = torch.full((px,), -1, device=dev, dtype=torch.int64)
    place[seen] = torch.arange(len(seen), device=dev)
    # every node x of the bound at depth z has g(x) = g(z) with g(x) = x - sum_j c_j / (x - t_j)
    t_all = zeros.to(dev)
    c_all = (vec[:, n - 1, :].to(dev) * b[n - 1][:, None]) ** 2
    lead = torch.ones(len(seen), device=dev, dtype=torch.float64)
    for v in b:
        lead = lead / (v * v)
    cols = torch.zeros((parts * px, 4), device=dev, dtype=torch.float64)

    def kernel(x, t, c, k2):  # K(x, x)
        d = [x - t[:, j] for j in range(n)]
        sq = torch.ones_like(x)
        for v in d:
            sq = sq * v * v
        for j in range(n):
            other = torch.ones_like(x)
            for i in range(n):
                if i != j:
                    other = other * d[i] * d[i]
            sq = sq + c[:, j] * other
        return k2 * sq

    for slot, z, dep, x in kept:
        for lo in range(0, len(z), 1 << 22):
            sl, zz, dd, xx = (v[lo:lo + (1 << 22)] for v in (slot.long(), z, dep, x))
            at = place[sl % px]
            on = at >= 0
            sl, zz, dd, xx, at = sl[on], zz[on], dd[on], xx[on], at[on]
            t, c, k2 = t_all[at], c_all[at], lead[at]
            goal = zz - (c / (zz[:, None] - t)).sum(dim=1)
            below = (t < zz[:, None]).sum(dim=1)
            frac = ETA / kernel(zz, t, c, k2)
            for i in range(n):  # the node in the gap below zero i, where z lies above that gap
                use = torch.nonzero(below > i).squeeze(1)
                if not len(use):
                    continue
                tu, cu, gu = t[use], c[use], goal[use]
                if i == 0:  # x = t_0 - y / (1 - y)
                    left, right = torch.zeros_like(gu), torch.ones_like(gu)
                else:
                    left, right = tu[:, i - 1].clone(), tu[:, i].clone()
                for _ in range(56):
                    mid = 0.5 * (left + right)
                    node = tu[:, 0] - mid / (1 - mid) if i == 0 else mid
                    high = node - (cu / (node[:, None] - tu)).sum(dim=1) > gu
                    if i == 0:
                        left, right = torch.where(high, mid, left), torch.where(high, right, mid)
                    else:
                        left, right = torch.where(high, left, mid), torch.where(high, mid, right)
                mid = 0.5 * (left + right)
                node = tu[:, 0] - mid / (1 - mid) if i == 0 else mid
                frac[use] += 1.0 / kernel(node, tu, cu, k2[use])
            trans = torch.exp(-mom[0][sl % px] * frac).clamp(0, 1)
            wgt = trans * -torch.expm1(-dd)
            e = xx.long().clamp(max=len(table) - 2)
            rgb = table[e, :3] + (table[e + 1, :3] - table[e, :3]) * (xx - e)[:, None]
            cols.index_add_(0, sl, wgt[:, None] * torch.cat([rgb, torch.ones_like(wgt)[:, None]], dim=1))
    return cols.reshape(parts, px, 4)
