"""Timed cases: what a program has this library do, through its public entry points.

A case is a dict of plain values.  Its ``kind`` says which entry points run:

* ``knn``        pg_knn: neighbour lists of recorded vertices
* ``edges``      pg_edges: aggregation weights and direct terms over given neighbour lists
* ``propagate``  pg_propagate: D iterations over a given weighted graph
* ``render``     a kept Renderer: the whole image (k nearest, or the cluster relation)
* ``grad``       one optimisation step: a taped render, a squared-error loss and pg_backward on the
                 tape, or (``autograd``) render_differentiable and its backward
* ``trace``      pg_trace: the instrumented path tracer
* ``batch``      a kept Batch plan (one graph launch) over independent scenes

The media, views and method settings are those of the repository's workloads (the small fBm cube, the
128^3 ball at 4 spp, the 512^3 cloud seen close up, the mixed batch).  Every input is made on the GPU from
the seed alone: a value-noise medium, then delta-tracked paths with their records, vectorised over the
paths with torch.  Weights and initial radiance that a case only reads are made with torch as well;
neighbour lists (whole numbers, the same for every correct search) come from pg_knn.
"""
import math

import torch
import torch.nn.functional as F

import paper_2404_11894_amd as pg

SUN = tuple(v / math.sqrt(0.3 ** 2 + 1.0 + 0.4 ** 2) for v in (0.3, 1.0, -0.4))
SUN_E = (2.0, 1.9, 1.7)
ENV_L = (0.25, 0.35, 0.5)
ENV_PDF = 1.0 / (4.0 * math.pi)
CAM, LOOK = (0.5, 0.5, -1.2), (0.5, 0.5, 0.5)

# The three media of the workloads: grid resolution, extinction maximum, fBm contrast and bias, soft ball
# radii (0, 0: the whole cube), albedo range, HG g, path depth, field of view.
MEDIA = {
    "tiny": dict(R=32, sigma=8.0, contrast=1.0, bias=0.0, r0=0.0, r1=0.0, lo=0.9, hi=0.9, g=0.5, depth=8, vfov=50.0),
    "mid": dict(R=128, sigma=32.0, contrast=2.0, bias=0.75, r0=0.42, r1=0.5, lo=0.95, hi=0.999, g=0.8, depth=64,
                vfov=20.0),
    "large": dict(R=256, sigma=64.0, contrast=2.0, bias=0.75, r0=0.0, r1=0.0, lo=0.999, hi=0.999, g=0.9, depth=128,
                  vfov=10.0),
}


def _case(name, kind, medium, width, height, spp, n, k, D, **more):
    c = dict(name=name, kind=kind, medium=medium, width=width, height=height, spp=spp, n=n, k=k, D=D)
    c.update(more)
    return c


def listed():
    return [
        # an interactive preview's iteration on the small cube: a few launches over 30k vertices
        _case("propagate_tiny", "propagate", "tiny", 64, 64, 4, 29011, 8, 8),
        # the iteration by itself, on a graph that a program built step by step and keeps
        _case("propagate_mid", "propagate", "mid", 257, 255, 4, 5000000, 16, 64),
        # neighbour lists of one full image, for a program with its own weights
        _case("knn_mid", "knn", "mid", 512, 512, 4, 20000001, 16, 0),
        # weights over given lists, an odd neighbour count, with volume emission
        _case("edges_mid", "edges", "mid", 256, 256, 3, 3800000, 13, 0, emit=True),
        # the smallest whole render: launch latency counts
        _case("render_tiny", "render", "tiny", 64, 64, 4, 29011, 8, 8),
        # the ordinary whole render, the converged radiance kept beside the image
        _case("render_mid", "render", "mid", 512, 512, 4, 20000000, 16, 64, lplus=True),
        # the headline: a dense cloud filling the image
        _case("render_large", "render", "large", 1024, 1024, 1, 64000000, 16, 128),
        # the paper's own neighbour relation
        _case("clusters_mid", "render", "mid", 512, 512, 4, 20000000, 16, 64, clusters=True),
        # a step of inverse rendering: tape with stored sums, gradients of grid, albedo and g
        _case("grad_mid", "grad", "mid", 256, 256, 4, 5000003, 16, 32, store_z=True, grid=64),
        # the same through autograd on a small crop, the settings left at their defaults
        _case("grad_small", "grad", "tiny", 61, 47, 3, 11003, 12, 10, autograd=True, grid=16),
        # the records of the ball traced on the device
        _case("trace_mid", "trace", "mid", 512, 512, 4, 20000000, 0, 0),
        # many independent scenes in one graph launch
        _case("batch_16", "batch", "tiny", 0, 0, 1, 0, 0, 0, scenes=16, lo=1e4, hi=1e6),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _drawn(*args, **more):
    c = _case("", *args, **more)
    del c["name"]
    return c


def draw(rng):
    kind = rng.choice(["propagate", "propagate", "knn", "knn", "edges", "edges", "render", "render", "clusters", "grad",
                       "trace", "batch"])
    if kind == "batch":
        return _drawn("batch", "tiny", 0, 0, 1, 0, 0, 0, scenes=rng.randint(3, 24), lo=1e4, hi=round(_log(rng, 1e5, 1e6)))
    medium = rng.choice(["tiny", "mid", "mid", "large"])
    spp = rng.choice([1, 1, 2, 3, 4])
    per = {"tiny": 1.9, "mid": 21.0, "large": 66.0}[medium]
    top = {"propagate": 6e6, "knn": 2e7, "edges": 8e6, "render": 2e7, "clusters": 2e7, "grad": 3e6, "trace": 2e7}[kind]
    n = round(_log(rng, 2e3, top))
    side = max(5.0, math.sqrt(n / (0.9 * per) / spp))
    aspect = math.exp(rng.uniform(-0.4, 0.4))
    w, h = max(3, round(side * aspect)), max(3, round(side / aspect))
    k = rng.choice([8, 16, 16, rng.randint(4, 24)])
    D = rng.choice([8, 16, rng.randint(1, 64), 64])
    more = {}
    if kind in ("render", "edges", "grad", "clusters") and rng.random() < 0.3:
        more["emit"] = True
    if kind in ("render", "clusters"):
        if rng.random() < 0.3:
            more["init"] = "zero"
        if rng.random() < 0.3:
            more["final_gather"] = 1
        more["lplus"] = rng.random() < 0.5
    if kind == "clusters":
        kind, more["clusters"] = "render", True
    if kind == "grad":
        more["grid"] = rng.choice([16, 32, 64])
        more["store_z"] = rng.random() < 0.6
        more["clusters"] = rng.random() < 0.2
        D = min(D, 32)
    if kind in ("knn", "edges", "trace"):
        D = 0
    return _drawn(kind, medium, w, h, spp, n, 0 if kind == "trace" else k, D, **more)


# ------------------------------------------------------------------ inputs ---

def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 2654435761 % (1 << 31) + 17)


def _noise(gen, R):
    """Value-noise fBm on an R^3 grid: four octaves from frequency 4, gain 1/2, in [0, 1]."""
    total, amp, f = torch.zeros(R, R, R, device="cuda"), 1.0, 4
    norm = 0.0
    for _ in range(4):
        lattice = torch.rand(1, 1, f + 1, f + 1, f + 1, generator=gen, device="cuda")
        total += amp * F.interpolate(lattice, size=(R, R, R), mode="trilinear", align_corners=True)[0, 0]
        norm += amp
        amp, f = amp * 0.5, f * 2
    return total / norm


def _medium(m, gen):
    """(extinction grid [z, y, x], albedo grid)"""
    R = m["R"]
    s = (0.5 + m["contrast"] * (_noise(gen, R) - 0.5) + m["bias"]).clamp_(0.0, 1.0)
    if m["r1"] > 0.0:
        a = (torch.arange(R, device="cuda") + 0.5) / R - 0.5
        rad = torch.sqrt(a[:, None, None] ** 2 + a[None, :, None] ** 2 + a[None, None, :] ** 2)
        t = ((rad - m["r0"]) / (m["r1"] - m["r0"])).clamp_(0.0, 1.0)
        s = s * (1.0 - t * t * (3.0 - 2.0 * t))
    alb = m["lo"] + (m["hi"] - m["lo"]) * torch.rand(R, R, R, generator=gen, device="cuda")
    return (m["sigma"] * s).contiguous(), alb.contiguous()


def _at(grid, p):
    R = grid.shape[0]
    i = (p * R).long().clamp_(0, R - 1)
    return grid.reshape(-1)[(i[:, 2] * R + i[:, 1]) * R + i[:, 0]]


def _unit(v):
    return v / v.norm(dim=1, keepdim=True)


def _hg_direction(t, g, gen):
    u = torch.rand(len(t), 2, generator=gen, device="cuda")
    if abs(g) < 1e-3:
        mu = 1.0 - 2.0 * u[:, 0]
    else:
        s = (1.0 - g * g) / (1.0 - g + 2.0 * g * u[:, 0])
        mu = (1.0 + g * g - s * s) / (2.0 * g)
    mu = mu.clamp_(-1.0, 1.0)
    st, phi = torch.sqrt((1.0 - mu * mu).clamp_(min=0.0)), 2.0 * math.pi * u[:, 1]
    helper = torch.zeros_like(t)
    helper[:, 0] = (t[:, 0].abs() < 0.7).float()
    helper[:, 1] = 1.0 - helper[:, 0]
    b1 = _unit(torch.linalg.cross(t, helper))
    b2 = torch.linalg.cross(t, b1)
    return _unit(mu[:, None] * t + (st * torch.cos(phi))[:, None] * b1 + (st * torch.sin(phi))[:, None] * b2)


def _sphere(n, gen):
    u = torch.rand(n, 2, generator=gen, device="cuda")
    z = 1.0 - 2.0 * u[:, 0]
    r, phi = torch.sqrt((1.0 - z * z).clamp_(min=0.0)), 2.0 * math.pi * u[:, 1]
    return _unit(torch.stack([r * torch.cos(phi), r * torch.sin(phi), z], 1))


def _exit(p, d):
    """Distance from p inside the unit cube to its boundary along d."""
    t = torch.where(d > 0, (1.0 - p) / d.clamp(min=1e-9), -p / d.clamp(max=-1e-9))
    return t.min(1).values.clamp_(min=0.0)


class _Scene:
    """Path-ordered records, as DevicePaths reads them."""


def _camera(width, height, vfov, gen, n, spp):
    pix = torch.arange(n, device="cuda") // spp
    u = torch.rand(n, 2, generator=gen, device="cuda")
    th = math.tan(0.5 * vfov * math.pi / 180.0)
    sx = (((pix % width) + u[:, 0]) / width * 2.0 - 1.0) * th * (width / height)
    sy = (1.0 - ((pix // width) + u[:, 1]) / height * 2.0) * th
    return _unit(torch.stack([sx, sy, torch.ones_like(sx)], 1))


def _scene(m, width, height, spp, n, seed, emit=False, keys=False):
    """Delta-tracked paths through the medium `m`, one per camera sample, with exactly n vertices in all: the
    paths' tails are cut evenly to that number (where there are fewer, the medium is made denser)."""
    for _ in range(12):
        s = _traced(m, width, height, spp, n, seed, emit, keys)
        if s is not None:
            return s
        m = dict(m, sigma=m["sigma"] * 1.15, depth=m["depth"] + m["depth"] // 8)
    raise ValueError("the view holds too few vertices for this case")


def _traced(m, width, height, spp, n, seed, emit, keys):
    gen = _generator(seed)
    sigma, alb = _medium(m, gen)
    P, maj, env = width * height * spp, float(m["sigma"]), torch.tensor(ENV_L, device="cuda")
    d = _camera(width, height, m["vfov"], gen, P, spp)
    o = torch.tensor(CAM, device="cuda")
    ta, tb = (0.0 - o) / d.where(d.abs() > 1e-9, torch.full_like(d, 1e-9)), (1.0 - o) / d.where(
        d.abs() > 1e-9, torch.full_like(d, 1e-9))
    t0, t1 = torch.minimum(ta, tb).max(1).values, torch.maximum(ta, tb).min(1).values
    hit = (t0 < t1) & (t0 > 0)
    pid = torch.nonzero(hit).squeeze(1)
    d = d[pid]
    p = (o + (t0[pid] + 1e-6)[:, None] * d).clamp_(0.0, 1.0)
    depth = torch.zeros(len(pid), dtype=torch.int64, device="cuda")
    escaped = ~hit
    got = []
    while len(pid):
        u = torch.rand(len(pid), 2, generator=gen, device="cuda")
        p = p + (-torch.log1p(-u[:, 0]) / maj)[:, None] * d
        inside = ((p >= 0.0) & (p <= 1.0)).all(1)
        escaped[pid[~inside]] = True
        pid, p, d, depth, u = pid[inside], p[inside], d[inside], depth[inside], u[inside]
        real = u[:, 1] * maj < _at(sigma, p)
        out = _hg_direction(d, m["g"], gen)
        got.append((pid[real], depth[real], p[real], d[real], out[real]))
        d = torch.where(real[:, None], out, d)
        depth = depth + real
        on = depth < m["depth"]
        pid, p, d, depth = pid[on], p[on], d[on], depth[on]
    pid, depth, p, d, out = (torch.cat([g[i] for g in got]) for i in range(5))
    del got
    count = torch.zeros(P, dtype=torch.int64, device="cuda")
    count.scatter_reduce_(0, pid, depth + 1, "amax")
    whole = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"), count.cumsum(0)])
    if len(pid) < n:
        return None
    s = _Scene()
    s.width, s.height, s.spp = width, height, spp
    s.path_offsets = whole * n // len(pid)
    kept = s.path_offsets[1:] - s.path_offsets[:-1]
    on = depth < kept[pid]
    pid, depth, p, d, out = pid[on], depth[on], p[on], d[on], out[on]
    at = s.path_offsets[pid] + depth
    N = n
    last = escaped & (count > 0) & (kept == count)
    s.pos, s.dir_in, s.dir_out = (torch.empty(N, 3, device="cuda") for _ in range(3))
    s.pos[at], s.dir_in[at], s.dir_out[at] = p, d, out
    del pid, depth, p, d, out, at
    s.albedo = _at(alb, s.pos)
    s.l_phase = torch.zeros(N, 3, device="cuda")
    s.l_phase[s.path_offsets[1:][last] - 1] = env
    s.e_cam = torch.where((escaped & (count == 0))[:, None], env, torch.zeros_like(env)).contiguous()
    here = _at(sigma, s.pos)
    sun = torch.tensor(SUN, device="cuda").expand(N, 3)

    def shadow(direction):   # transmittance as shadow rays report it: spread over decades, often exactly 0
        x = torch.rand(N, 2, generator=gen, device="cuda")
        return torch.exp(-here * _exit(s.pos, direction) * x[:, 0]) * (x[:, 1] < 0.7)

    s.l_sun = shadow(sun)[:, None] * torch.tensor(SUN_E, device="cuda")
    s.dir_env = _sphere(N, gen)
    s.l_env = shadow(s.dir_env)[:, None] * env
    if emit:
        r2 = ((s.pos - 0.5) ** 2).sum(1)
        s.l_emit = ((1.0 - s.albedo) * (1.0 - r2 / 0.0625).clamp_(min=0.0) ** 2)[:, None] * torch.tensor(
            (3.0, 2.0, 1.0), device="cuda")
    if keys:
        s.cluster_key = torch.randint(-2 ** 31, 2 ** 31 - 1, (N,), generator=gen, device="cuda",
                                      dtype=torch.int64).to(torch.int32)
    return s


def _of_case(case, seed, **more):
    m = MEDIA[case["medium"]]
    return _scene(m, case["width"], case["height"], case["spp"], case["n"], seed, emit=bool(case.get("emit")), **more)


def _params(case, **more):
    return pg.params(k=case["k"], D=case["D"], g=MEDIA[case["medium"]]["g"], init=case.get("init", "pt"),
                     final_gather=case.get("final_gather", 0), **more)


def _hg(u, g):
    """HG density over u = 1 - cos."""
    return (1.0 - g * g) / (4.0 * math.pi) * ((1.0 - g) ** 2 + 2.0 * g * u) ** -1.5


def _u(a, b):
    return 0.5 * ((a - b) ** 2).sum(-1)


def _weights(s, col, K, g, dtype=torch.float32, chunk=1 << 18):
    """Per row: the indirect weights, the direct weights of the phase and emitter samples, and the terms
    b, d_pt and r, from the definition of the aggregation operators."""
    N = len(s.pos)
    sun = torch.tensor(SUN, dtype=dtype, device="cuda")
    parts = []
    for a in range(0, N, chunk):
        j = col[a * K:(a + chunk) * K].long().reshape(-1, K)
        t, w, we, ls, le, lp = (getattr(s, n)[j].to(dtype) for n in
                                ("dir_in", "dir_out", "dir_env", "l_sun", "l_env", "l_phase"))
        ti = t[:, :1]
        mp = _hg(_u(t[:, None, :, :], w[:, :, None, :]), g).sum(2)
        me = _hg(_u(t[:, None, :, :], we[:, :, None, :]), g).sum(2) + K * ENV_PDF
        rw, re = _hg(_u(ti, w), g), _hg(_u(ti, we), g)
        w_ind, w_ph, w_env = rw / mp, rw / (mp + K * ENV_PDF), re / me
        rs = _hg(_u(ti[:, 0], sun), g)
        d_agg = rs[:, None] * ls.mean(1) + (w_env[..., None] * le + w_ph[..., None] * lp).sum(1)
        al = s.albedo[a:a + chunk].to(dtype)
        b = al[:, None] * d_agg
        if getattr(s, "l_emit", None) is not None:
            b = b + s.l_emit[a:a + chunk].to(dtype)
        d_pt = (rs[:, None] * ls[:, 0] + (re[:, 0] / (re[:, 0] + ENV_PDF))[:, None] * le[:, 0]
                + (rw[:, 0] / (rw[:, 0] + ENV_PDF))[:, None] * lp[:, 0])
        parts.append((w_ind, w_ph, w_env, b, d_pt))
    return tuple(torch.cat([q[i] for q in parts]) for i in range(5))


def _successors(s):
    """Path-order id of each vertex's successor, and whether there is one."""
    N = len(s.pos)
    end = torch.zeros(N, dtype=torch.bool, device="cuda")
    off = s.path_offsets
    end[off[1:][off[1:] > off[:-1]] - 1] = True
    return torch.arange(1, N + 1, device="cuda").clamp_(max=N - 1), ~end


def _path_estimate(s, d_pt, dtype):
    """The path tracer's own incoming radiance (g = g_s, so the continuation ratio is 1), by recursive
    doubling of the affine maps L(v) = e_u + albedo_u (d_pt_u + L(u))."""
    succ, has = _successors(s)
    al = s.albedo.to(dtype)
    A = al[:, None] * d_pt
    if getattr(s, "l_emit", None) is not None:
        A = A + s.l_emit.to(dtype)
    A = torch.where(has[:, None], A[succ], torch.zeros_like(A))   # v's map takes the value at its successor
    B = torch.where(has, al[succ], torch.zeros_like(al))
    nxt, steps = succ.clone(), int((s.path_offsets[1:] - s.path_offsets[:-1]).max())
    n = 1
    while n < steps:
        A = A + B[:, None] * A[nxt]
        B = B * B[nxt]
        nxt = nxt[nxt]
        n *= 2
    return A


# ----------------------------------------------------------------- prepare ---

def _batch_scenes(case, seed):
    import random
    rng = random.Random(int(case["scenes"]) * 7919 + int(case["hi"]))
    out = []
    for i in range(case["scenes"]):
        m = dict(MEDIA["tiny"], sigma=rng.uniform(6.0, 24.0), g=rng.uniform(-0.3, 0.9), vfov=40.0)
        m["lo"] = m["hi"] = rng.uniform(0.8, 0.999)
        k, D = rng.randint(8, 16), rng.randint(16, 64)
        m["depth"] = D
        n = round(_log(rng, case["lo"], case["hi"]))
        per = 0.36 * m["sigma"]
        side = max(8, round(math.sqrt(n / per)))
        out.append((m, side, n, k, D, int(seed) * 64 + i))
    return out


def prepare(case, seed):
    kind = case["kind"]
    if kind == "trace":
        # the path geometry belongs to the case (its record count is the outputs' shape); the seed draws the
        # albedo and the light colours
        m, gen = MEDIA[case["medium"]], _generator(seed)
        sigma, _ = _medium(m, _generator(case["width"] + case["height"]))
        R = m["R"]
        alb = m["lo"] - 0.05 + (m["hi"] - m["lo"] + 0.05) * torch.rand(R, R, R, generator=gen, device="cuda")
        tint = (0.8 + 0.4 * torch.rand(2, 3, generator=gen, device="cuda")).tolist()
        settings = dict(R=R, width=case["width"], height=case["height"], spp=case["spp"], max_depth=m["depth"],
                        albedo_const=m["lo"], g=m["g"], cam_pos=CAM, look_at=LOOK, vfov_deg=m["vfov"], sun_dir=SUN,
                        sun_E=[a * b for a, b in zip(SUN_E, tint[0])], env_L=[a * b for a, b in zip(ENV_L, tint[1])],
                        seed=case["n"])
        return dict(kind=kind, settings=settings, sigma=sigma, albedo=alb, majorant=float(m["sigma"]))
    if kind == "batch":
        paths, qs = [], []
        for m, side, n, k, D, sd in _batch_scenes(case, seed):
            paths.append(pg.DevicePaths(_scene(m, side, side, 1, n, sd)))
            qs.append(pg.params(k=k, D=D, g=m["g"]))
        return dict(kind=kind, plan=pg.Batch(paths, qs))
    clusters = bool(case.get("clusters"))
    s = _of_case(case, seed, keys=clusters)
    flags = pg.PG_FLAG_CLUSTERS if clusters else 0
    if kind == "grad":
        gen = _generator(seed + 1)
        R = case["grid"]
        grid = 0.95 + 0.049 * torch.rand(R, R, R, generator=gen, device="cuda")
        target = 0.6 * torch.rand(case["height"], case["width"], 3, generator=gen, device="cuda")
        if case.get("autograd"):
            return dict(kind="autograd", paths=pg.DevicePaths(s), q=_params(case, flags=flags), target=target,
                        grid=grid.requires_grad_(), g=torch.tensor(MEDIA[case["medium"]]["g"], requires_grad=True))
        paths = pg.DevicePaths(s, albedo_grid=grid)
        flags |= pg.PG_FLAG_TAPE | (pg.PG_FLAG_STORE_Z if case.get("store_z") else 0)
        return dict(kind=kind, paths=paths, target=target, renderer=pg.Renderer(paths, _params(case, flags=flags)))
    paths = pg.DevicePaths(s)
    if kind == "knn":
        return dict(kind=kind, paths=paths, k=case["k"])
    if kind == "render":
        graph = dict(lplus=torch.empty(paths.n_vertices, 3, device="cuda")) if case.get("lplus") else None
        return dict(kind=kind, renderer=pg.Renderer(paths, _params(case, flags=flags)), graph=graph)
    row_ptr, col = pg.pg_knn(paths, case["k"])
    q = _params(case)
    if kind == "edges":
        return dict(kind=kind, paths=paths, q=q, row_ptr=row_ptr, col=col)
    K = min(case["k"], paths.n_vertices)
    w, _, _, b, d_pt = _weights(s, col, K, MEDIA[case["medium"]]["g"])
    x0 = _path_estimate(s, d_pt, torch.float32)
    return dict(kind=kind, paths=paths, q=q, row_ptr=row_ptr, col=col, w=w.reshape(-1).contiguous(), b=b.contiguous(),
                x0=x0.contiguous())


def run(state):
    kind = state["kind"]
    if kind == "knn":
        return pg.pg_knn(state["paths"], state["k"])
    if kind == "edges":
        return pg.pg_edges(state["paths"], state["q"], state["row_ptr"], state["col"])
    if kind == "propagate":
        return pg.pg_propagate(state["paths"], state["q"], state["row_ptr"], state["col"], state["w"], state["b"],
                               state["x0"].clone())
    if kind == "render":
        image = state["renderer"](graph=state["graph"])
        return [image, state["graph"]["lplus"]] if state["graph"] else image
    if kind == "grad":
        r = state["renderer"]
        image = r()
        out = pg.pg_backward(state["paths"], r.q, 2.0 * (image - state["target"]), grad_albedo=True,
                             workspace=(r.ws, r.ws_bytes))
        return dict(out, image=image)
    if kind == "autograd":
        image = pg.render_differentiable(state["paths"], state["q"], state["grid"], state["g"])
        loss = ((image - state["target"]) ** 2).sum()
        grid, g = torch.autograd.grad(loss, (state["grid"], state["g"]))
        return dict(image=image.detach(), grad_grid=grid, grad_g=g)
    if kind == "trace":
        r = pg.pg_trace(state["settings"], state["sigma"], state["albedo"], majorant=state["majorant"])
        return {n: getattr(r, n) for n in ("path_offsets", "pos", "dir_in", "dir_out", "albedo", "l_sun", "dir_env",
                                           "l_env", "l_phase", "e_cam")}
    return state["plan"]()


# -------------------------------------------------------------------- work ---

def work(case):
    """Bytes: every array of the call read or written once; where the call iterates, the operator (a 4-byte id
    and a 4-byte weight per edge), the constants and both radiance vectors once an iteration."""
    kind, K, D = case["kind"], case["k"], case["D"]
    if kind == "batch":
        by = fl = 0.0
        for m, side, n, k, d, _ in _batch_scenes(case, 0):
            by += n * (88 + d * (8 * k + 68)) + 12 * side * side
            fl += n * (d * 6 * k + 28 * k * k)
        return dict(bytes=by, flops=fl)
    P, N = case["width"] * case["height"] * case["spp"], case["n"]
    image = 12.0 * case["width"] * case["height"]
    if kind == "trace":
        return dict(bytes=88 * N + 20 * P, flops=1000 * N)
    if kind == "knn":
        return dict(bytes=N * (12 + 8 + 4 * K), flops=N * 8 * 4 * K)
    if kind == "edges":
        return dict(bytes=N * (76 + 4 * K + 12 * K + 36 + (12 if case.get("emit") else 0)), flops=N * 28 * K * K)
    if kind == "propagate":
        return dict(bytes=D * N * (8 * K + 68), flops=D * N * 6 * K)
    row = 80 if case.get("clusters") else 8 * K + 68
    forward = dict(bytes=N * (88 + D * row) + 20 * P + image, flops=N * (D * 6 * K + 28 * K * K))
    if kind == "grad":   # the reverse iteration reads the operator and the adjoint vectors once more
        return dict(bytes=2 * forward["bytes"] + 4.0 * case["grid"] ** 3, flops=2 * forward["flops"])
    return forward


# ------------------------------------------------------------------- exact ---

def _neighbours(pos, K):
    """The K nearest by (squared distance of the 20-bit quantised positions, id), the vertex first."""
    N = len(pos)
    q = (pos * 1048576.0).floor().clamp_(0, 1048575).to(torch.int64)
    ids = torch.arange(N, device="cuda")
    rows = []
    for a in range(0, N, 1024):
        dd = torch.zeros(min(1024, N - a), N, dtype=torch.int64, device="cuda")
        for ax in range(3):
            dd += (q[a:a + 1024, ax:ax + 1] - q[None, :, ax]) ** 2
        key = ((dd + 1) << 20) | ids
        key[torch.arange(len(dd), device="cuda"), ids[a:a + 1024]] = 0
        idx = key.topk(K, dim=1, largest=False, sorted=True).indices
        rows.append(idx)
    return torch.cat(rows)


def _trilerp(grid, pos):
    R = grid.shape[0]
    u = R * pos.double() - 0.5
    f0 = u.floor()
    f, i0 = u - f0, f0.long()
    out = 0.0
    for c in range(8):
        w, idx = 1.0, []
        for ax in range(3):
            bit = (c >> ax) & 1
            idx.append((i0[:, ax] + bit).clamp(0, R - 1))
            w = w * (f[:, ax] if bit else 1.0 - f[:, ax])
        out = out + w * grid[idx[2], idx[1], idx[0]]
    return out


def _render64(s, case, grid=None, g=None):
    """The whole render in 64 bits, differentiable in the albedo grid and the receivers' g."""
    N, D = len(s.pos), case["D"]
    K = min(case["k"], N)
    gs = torch.tensor(MEDIA[case["medium"]]["g"], dtype=torch.float32).double().item()   # as the call holds it
    g = gs if g is None else g
    j = _neighbours(s.pos, K)
    al = s.albedo.double() if grid is None else _trilerp(grid, s.pos)
    t, w, we, ls, le, lp = (getattr(s, n).double() for n in ("dir_in", "dir_out", "dir_env", "l_sun", "l_env",
                                                             "l_phase"))
    sun = torch.tensor(SUN, dtype=torch.float32, device="cuda").double()
    pe = torch.tensor(ENV_PDF, dtype=torch.float32).double().item()
    em = s.l_emit.double() if getattr(s, "l_emit", None) is not None else torch.zeros_like(ls)
    tj, wj, wej = t[j], w[j], we[j]
    mp, me = torch.zeros(N, K, dtype=torch.float64, device="cuda"), torch.zeros(N, K, dtype=torch.float64, device="cuda")
    for l in range(K):
        mp += _hg(_u(tj[:, l:l + 1], wj), gs)
        me += _hg(_u(tj[:, l:l + 1], wej), gs)
    rw, re = _hg(_u(t[:, None], wj), g), _hg(_u(t[:, None], wej), g)
    W = rw / mp
    rs = _hg(_u(t, sun), g)
    d_agg = rs[:, None] * ls[j].mean(1) + ((re / (me + K * pe))[..., None] * le[j]
                                           + (rw / (mp + K * pe))[..., None] * lp[j]).sum(1)
    b = em + al[:, None] * d_agg
    pw, pq = _hg(_u(t, w), gs), _hg(_u(t, we), gs)
    d_pt = (rs[:, None] * ls + (re[:, 0] / (pq + pe))[:, None] * le + (rw[:, 0] / (pw + pe))[:, None] * lp)
    r = rw[:, 0] / pw
    succ, has = _successors(s)
    A = em + (al[:, None] * d_pt if case.get("init", "pt") == "pt" else 0.0)
    B = al * r if case.get("init", "pt") == "pt" else torch.zeros_like(al)
    x = torch.zeros_like(ls)
    for _ in range(int((s.path_offsets[1:] - s.path_offsets[:-1]).max())):
        x = torch.where(has[:, None], A[succ] + B[succ, None] * x[succ], torch.zeros_like(x))
    for _ in range(D):
        y = b + al[:, None] * (W[..., None] * x[j]).sum(1)
        x = torch.where(has[:, None], y[succ], torch.zeros_like(y))
    off = s.path_offsets
    full = off[1:] > off[:-1]
    v0 = off[:-1].clamp(max=N - 1)
    inner = (W[v0][..., None] * x[j[v0]]).sum(1) if not case.get("final_gather") else r[v0, None] * x[v0]
    o = torch.where(full[:, None], em[v0] + al[v0, None] * (d_pt[v0] + inner), torch.zeros(3, dtype=torch.float64,
                                                                                         device="cuda"))
    image = (s.e_cam.double() + o).reshape(s.height, s.width, s.spp, 3).mean(2)
    return image, x


def exact(case, seed):
    kind = case["kind"]
    if kind in ("knn", "trace", "batch") or case.get("clusters"):
        return None   # whole numbers, or decisions (accepted flights, cluster splits) that have no 64-bit value
    if kind in ("edges", "propagate"):
        s = _of_case(case, seed)
        if kind == "edges":
            st = prepare(case, seed)
            g = torch.tensor(MEDIA[case["medium"]]["g"], dtype=torch.float32).double().item()
            K = min(case["k"], len(s.pos))
            w, wp, we, b, d_pt = _weights(s, st["col"], K, g, torch.float64, 1 << 17)
            x0 = _path_estimate(s, d_pt, torch.float64)
            return dict(w_ind=w.reshape(-1), w_ph=wp.reshape(-1), w_env=we.reshape(-1), b=b, d_pt=d_pt, lplus0=x0)
        st = prepare(case, seed)
        K = min(case["k"], len(s.pos))
        succ, has = _successors(s)
        x, b, al = st["x0"].double(), st["b"].double(), s.albedo.double()
        w, j = st["w"].reshape(-1, K), st["col"].reshape(-1, K).long()
        for _ in range(case["D"]):
            z = torch.zeros_like(x)
            for l in range(K):
                z += w[:, l:l + 1].double() * x[j[:, l]]
            y = b + al[:, None] * z
            x = torch.where(has[:, None], y[succ], torch.zeros_like(y))
        return x
    if case["n"] > 60000:
        return None   # the neighbour search by its definition would take too long
    s = _of_case(case, seed)
    if kind == "render":
        image, x = _render64(s, case)
        return [image, x] if case.get("lplus") else image
    st = prepare(case, seed)
    grid = (st["grid"].detach() if case.get("autograd") else st["paths"].albedo_grid).double().requires_grad_()
    g = torch.tensor(MEDIA[case["medium"]]["g"], dtype=torch.float32, device="cuda").double().requires_grad_()
    image, _ = _render64(s, case, grid, g)
    gi = 2.0 * (image.detach() - st["target"].double())
    ggrid, gg = torch.autograd.grad((image * gi).sum(), (grid, g))
    out = dict(image=image.detach(), grad_grid=ggrid, grad_g=gg if case.get("autograd") else gg.reshape(1))
    if not case.get("autograd"):
        out["grad_albedo"] = None
    return out

