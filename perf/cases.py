"""Performance cases of the library: what its users have it do, through the
Python binding (renders, the density octree, the learned density, densities
over a point set), from the smallest calls to the largest.

A case is a dict of plain values; prepare() builds what a program holds
before the call, run() is one pass, work() the traffic and arithmetic a pass
cannot do without and exact() the same outputs from plain torch in 64 bits
where they are a closed computation.

Renders with the octree's density trace conventional light photons too: its
splits race with its deposits, so the fluxes of a few photons, and with them
the image, differ from run to run; light photons bound those photons' weight
(balance heuristic), which a frame of the room's size averages out.  The
other density providers, and path tracing without photons, give the same
image twice up to the order of additions.
"""
import ctypes
import math

import numpy as np
import torch

import neb_inputs
from paper_1909_00573_amd import neb

DENSITIES = {"robust": neb.DENSITY_OCTREE_ROBUST, "radius": neb.DENSITY_RADIUS, "knn": neb.DENSITY_KNN}
# density radii: one to two merge radii of the scene
RADII = {"tiny_box": 0.02, "room": 0.04, "city": 0.4, "box_room": 0.0124}

# learned density: widths and the flat parameter layout of the binding
ENC, WIDTH = 80, 64
MU, SIGMA = 7.5, 1.4  # log density of a room's NEE vertices: mean and spread


def listed():
    return [
        # the smallest whole job: a 64 x 64 preview, bound by launches and latency
        dict(name="tiny_box", kind="render", scene="tiny_box", width=64, height=64, maxlen=5, spp=4, density="radius",
             light_photons=0, nee_radius=0.0, detail=0, lights=0),
        # the flagship room at full size with the default (robust octree) density
        dict(name="room", kind="render", scene="room", width=512, height=512, maxlen=8, spp=8, density="robust",
             light_photons=262144, nee_radius=0.0, detail=5, lights=0),
        # plain path tracing of the same room: camera paths and NEE, no photons
        dict(name="room_paths", kind="render", scene="room", width=512, height=512, maxlen=8, spp=16, density="none",
             light_photons=0, nee_radius=0.0, detail=5, lights=0),
        # an odd, wide frame with photons from the nearest-neighbour density
        dict(name="room_knn", kind="render", scene="room", width=401, height=227, maxlen=8, spp=4, density="knn",
             light_photons=0, nee_radius=0.0, detail=4, lights=0),
        # the scale case: a million triangles, a thousand point lights, GGX and mirror surfaces
        dict(name="city", kind="render", scene="city", width=1024, height=1024, maxlen=10, spp=2, density="radius",
             light_photons=0, nee_radius=0.0, detail=288, lights=1024),
        # many scenes of uneven size in one context
        dict(name="batch", kind="batch", scenes=12, smallest=64, largest=320, tris=6000, lights=40, spp=4,
             density="radius"),
        # one frame's learned densities: every vertex slot of the room
        dict(name="mlp_frame", kind="infer", n=1835008),
        # a handful of learned densities: one call's latency
        dict(name="mlp_few", kind="infer", n=1001),
        # learned density, training: Adam steps of the default batch and the updated weights
        dict(name="mlp_train", kind="train", n=65536, steps=8),
        # one iteration of the octree on a grown tree: clear, deposits, robust densities at the deposits
        dict(name="octree", kind="octree", n=1000003, grown=60000, iteration=250, robust=True),
        # k nearest neighbours over a point set, through the call that allocates its own grid
        dict(name="knn", kind="points", n=200000, queries=200000, density="knn", radius=0.004, k=8, alloc=True),
        # a small fixed-radius count without allocation (a serving loop)
        dict(name="radius_few", kind="points", n=3001, queries=3001, density="radius", radius=0.05, k=8,
             alloc=False),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["render", "render", "render", "batch", "infer", "train", "octree", "points"])
    if kind == "render":
        scene = rng.choice(["tiny_box", "room", "room", "city"])
        density = rng.choice(["robust", "radius", "knn", "none"]) if scene == "room" else rng.choice(
            ["radius", "knn", "none"])
        w = _log_int(rng, 400, 640) if density == "robust" else _log_int(rng, 48, 640)
        h = max(32, int(w * rng.uniform(0.7, 1.1)))
        recycle = scene == "room" and density == "none" and rng.random() < 0.5
        return dict(kind="render", scene=scene, width=w, height=h, maxlen=rng.randint(4, 9),
                    spp=2 if w * h > 100000 else rng.randint(2, 8), density=density,
                    light_photons=262144 if density == "robust" else 0, nee_radius=0.02 if recycle else 0.0,
                    detail={"tiny_box": 0, "room": rng.randint(2, 5), "city": _log_int(rng, 12, 200)}[scene],
                    lights=_log_int(rng, 16, 1024) if scene == "city" else 0)
    if kind == "batch":
        lo = _log_int(rng, 32, 128)
        return dict(kind="batch", scenes=rng.randint(2, 16), smallest=lo, largest=lo + _log_int(rng, 16, 160),
                    tris=_log_int(rng, 1500, 6000), lights=_log_int(rng, 4, 128), spp=rng.randint(2, 4),
                    density=rng.choice(["radius", "none"]))
    if kind == "infer":
        return dict(kind="infer", n=_log_int(rng, 17, 1835008))
    if kind == "train":
        return dict(kind="train", n=_log_int(rng, 256, 131072), steps=rng.randint(2, 8))
    if kind == "octree":
        return dict(kind="octree", n=_log_int(rng, 1000, 2000000), grown=_log_int(rng, 1000, 60000), iteration=250,
                    robust=rng.random() < 0.6)
    n = _log_int(rng, 500, 400000)
    density = rng.choice(["radius", "knn"])
    return dict(kind="points", n=n, queries=_log_int(rng, 500, 400000), density=density,
                radius=round(min(0.2, rng.uniform(1.5, 4.0) / math.sqrt(n)), 6), k=rng.randint(2, 16),
                alloc=rng.random() < 0.5)


# --------------------------------------------------------------------------
# inputs, from the seed alone
# --------------------------------------------------------------------------
def _rng(seed, device="cuda"):
    return torch.Generator(device=device).manual_seed(int(seed))


def _surface_points(n, seed, device="cuda"):
    """Points on the surfaces of a unit scene (two axis-aligned planes, a
    tilted one) and a dense ball around its centre, with their normals."""
    g = _rng(seed, device)
    uv = torch.rand(n, 2, generator=g, device=device) * 0.9 + 0.05
    which = torch.randint(0, 4, (n,), generator=g, device=device)
    ball = torch.randn(n, 3, generator=g, device=device)
    u, v = uv[:, 0], uv[:, 1]
    tilt = torch.stack([u, v, 0.2 + 0.5 * u + 0.1 * v], 1)
    planes = [torch.stack([u, torch.full_like(u, 0.3), v], 1), torch.stack([torch.full_like(u, 0.71), u, v], 1), tilt]
    ball = ball / ball.norm(dim=1, keepdim=True)
    normals = [torch.tensor(x, device=device) for x in ([0.0, 1.0, 0.0], [1.0, 0.0, 0.0])]
    tn = torch.tensor([-0.5, -0.1, 1.0], device=device)
    normals.append(tn / tn.norm())
    p, nrm = 0.5 + 0.12 * ball, ball.clone()
    for k in range(3):
        p = torch.where((which == k)[:, None], planes[k], p)
        nrm = torch.where((which == k)[:, None], normals[k], nrm)
    return p.contiguous(), nrm.contiguous()


def _weights(seed):
    """He-uniform initial parameters in the binding's layout (W1, b1, W2, b2,
    W3, b3, w4, b4), biases small."""
    r = np.random.default_rng(seed)

    def w(n, fan):
        return r.uniform(-1, 1, n) * math.sqrt(6.0 / fan)

    def b(n):
        return r.uniform(-0.05, 0.05, n)
    return np.concatenate([w(ENC * WIDTH, ENC), b(WIDTH), w(WIDTH * WIDTH, WIDTH), b(WIDTH), w(WIDTH * WIDTH, WIDTH),
                           b(WIDTH), w(WIDTH, WIDTH), b(1)]).astype(np.float32)


def _log_rho(p, n, seed, device="cuda"):
    """A smooth log density with the counting noise of an octree's leaves."""
    g = _rng(seed + 1, device)
    return (MU + SIGMA * (torch.sin(5 * p[:, 0]) + torch.cos(7 * p[:, 1]) * p[:, 2] + 0.3 * n[:, 1])
            + 0.3 * torch.randn(p.shape[0], generator=g, device=device)).contiguous()


def _scene(case, seed):
    kw = dict(width=case["width"], height=case["height"], spp=case["spp"], max_path_len=case["maxlen"], seed=seed)
    if case["scene"] == "tiny_box":
        return neb_inputs.tiny_box(**kw)
    if case["scene"] == "room":
        return neb_inputs.room(glass_subdiv=case["detail"], **kw)
    lots = case["detail"]
    return neb_inputs.city_block(lots=lots, n_lights=case["lights"], octree_capacity=1 << (24 if lots > 100 else 20),
                                 torus_quads=(200, 125) if lots > 100 else (24, 12), **kw)


def _settings(case):
    if case["density"] == "none":
        return dict(flags=neb.FLAG_NO_PHOTONS)
    return dict(density_mode=DENSITIES[case["density"]])


def _batch_sizes(case, seed):
    r = np.random.default_rng(seed)
    n = case["scenes"]
    res = [case["smallest"] + (case["largest"] - case["smallest"]) * i // (n - 1) for i in range(n)]
    tris = np.exp(r.uniform(math.log(1000), math.log(case["tris"]), n)).astype(int)
    lights = r.integers(1, case["lights"] + 1, n)
    return [(int(t), int(min(lt, max(1, (t - 12) // 80))), int(s)) for t, lt, s in zip(tris, lights, res)]


def prepare(case, seed):
    kind = case["kind"]
    if kind == "render":
        over = dict(light_photons=case["light_photons"], nee_radius=case["nee_radius"])
        if case["density"] in ("radius", "knn"):
            over["density_radius"] = RADII[case["scene"]]
        return dict(kind=kind, spp=case["spp"], r=neb.Renderer(_scene(case, seed), **_settings(case), **over))
    if kind == "batch":
        scenes = [neb_inputs.box_room(n_tris=t, n_lights=lt, res=s, spp=case["spp"], seed=seed, scene_id=i)
                  for i, (t, lt, s) in enumerate(_batch_sizes(case, seed))]
        per = [dict(density_radius=RADII["box_room"]) for _ in scenes]
        r = neb.BatchRenderer(scenes, per_scene=per, **_settings(case))
        r.reset()  # uploads the scenes
        return dict(kind=kind, spp=case["spp"], r=r)
    if kind == "infer":
        p, n = _surface_points(case["n"], seed)
        m = neb.Mlp(init=_weights(seed), max_batch=16)
        m.set_normalization(MU, SIGMA)
        return dict(kind=kind, m=m, p=p, n=n)
    if kind == "train":
        p, n = _surface_points(case["n"] * case["steps"], seed)
        t = _log_rho(p, n, seed)
        m = neb.Mlp(init=_weights(seed), max_batch=case["n"])
        m.set_normalization(MU, SIGMA)
        return dict(kind=kind, m=m, batches=[tuple(a[k * case["n"]:(k + 1) * case["n"]] for a in (p, n, t))
                                             for k in range(case["steps"])])
    if kind == "octree":
        o = neb.DeviceOctree(np.zeros(3, np.float32), np.ones(3, np.float32), 1 << 20)
        grow, _ = _surface_points(case["grown"], seed + 7)
        o.increment(grow, single_thread=True)  # the listed order: the same tree every time
        p, n = _surface_points(case["n"], seed)
        return dict(kind=kind, o=o, p=p, n=n, iteration=case["iteration"], robust=case["robust"])
    p, _ = _surface_points(case["n"], seed)
    q, _ = _surface_points(case["queries"], seed + 3)
    q[::2] = p[torch.arange(q[::2].shape[0], device=q.device) % p.shape[0]]
    return dict(kind=kind, p=p, q=q, mode=DENSITIES[case["density"]], radius=case["radius"], k=case["k"],
                alloc=case["alloc"], out=torch.empty(case["queries"], device="cuda"))


def run(s):
    kind = s["kind"]
    if kind in ("render", "batch"):
        r = s["r"]
        r.reset()
        r.render(s["spp"])
        return [r.image(i) for i in range(len(r.scenes))]
    if kind == "infer":
        return s["m"].infer(s["p"], s["n"])
    if kind == "train":
        for p, n, t in s["batches"]:
            s["m"].train_step(p, n, t, lr=2e-3)
        return s["m"].params()
    if kind == "octree":
        o = s["o"]
        o.clear_counters()
        o.set_iteration(s["iteration"])
        o.increment(s["p"])
        return o.density(s["p"], s["n"], robust=s["robust"])
    if s["alloc"]:
        return neb.point_density(s["p"], s["q"], s["mode"], s["radius"], s["k"])
    return neb.point_density_noalloc(s["p"], s["q"], s["mode"], s["radius"], s["k"], s["out"])


# --------------------------------------------------------------------------
# work a pass cannot do without
# --------------------------------------------------------------------------
def _render_work(pixels, spp, maxlen, tris, photons, light_photons):
    """Every pixel's image written once; per iteration the view vertices (64
    bytes, on average two thirds of the path length deep) written and read
    once, and the geometry (one 128-byte node and one 48-byte triangle of
    two) read once.  A ray takes about log4(triangles) + 3 node visits of
    four box tests (20 operations each) and three triangle tests (60)."""
    depth = max(1.0, 2.0 * maxlen / 3.0)
    vertices = pixels * depth
    rays = pixels * depth + vertices + ((vertices * 0.5 * depth) if photons else 0) + light_photons * depth
    visits = math.log(max(tris, 4), 4) + 3
    return (12.0 * pixels + spp * (128.0 * vertices + 88.0 * tris), spp * rays * (80.0 * visits + 180.0))


def work(case):
    kind = case["kind"]
    if kind == "render":
        tris = {"tiny_box": 334, "room": 3400 + 20 * 4 ** case["detail"],
                "city": 12 * case["detail"] ** 2 + (50000 if case["detail"] > 100 else 576)}[case["scene"]]
        b, f = _render_work(case["width"] * case["height"], case["spp"], case["maxlen"], tris,
                            case["density"] != "none", case["light_photons"])
        return {"bytes": b, "flops": f}
    if kind == "batch":
        side2 = (case["smallest"] ** 2 + case["smallest"] * case["largest"] + case["largest"] ** 2) / 3.0
        tris = (case["tris"] - 1000) / math.log(case["tris"] / 1000)
        b, f = _render_work(side2, case["spp"], 8, tris, case["density"] != "none", 0)
        return {"bytes": b * case["scenes"], "flops": f * case["scenes"]}
    layers = 2.0 * (78 * WIDTH + 2 * WIDTH * WIDTH + WIDTH)
    if kind == "infer":
        return {"bytes": 28.0 * case["n"] + 4.0 * neb.MLP_PARAMS, "flops": layers * case["n"]}
    if kind == "train":
        return {"bytes": (28.0 * case["n"] + 24.0 * neb.MLP_PARAMS) * case["steps"],
                "flops": 3.0 * layers * case["n"] * case["steps"]}
    if kind == "octree":
        # positions twice, normals and densities once, a node word updated per
        # deposit; per probe about 60 operations of the plane's area
        return {"bytes": 44.0 * case["n"], "flops": case["n"] * (300.0 if case["robust"] else 60.0)}
    ball = min(case["n"], case["n"] * 4.0 * case["radius"] ** 2)  # points a ball on a plane holds
    return {"bytes": 12.0 * case["n"] + 16.0 * case["queries"], "flops": 8.0 * ball * case["queries"]}


# --------------------------------------------------------------------------
# the same outputs in 64 bits
# --------------------------------------------------------------------------
def _model64(seed):
    w = torch.from_numpy(_weights(seed).astype(np.float64)).cuda()
    out, at = [], 0
    for n in (ENC * WIDTH, WIDTH, WIDTH * WIDTH, WIDTH, WIDTH * WIDTH, WIDTH, WIDTH, 1):
        out.append(w[at:at + n].clone())
        at += n
    return out


def _encode64(p, n):
    c = torch.cat([p, n], 1).double()
    x = [c]
    for i in range(6):
        for o in range(6):
            a = c[:, i] * (2.0 ** o * math.pi)
            x += [torch.sin(a)[:, None], torch.cos(a)[:, None]]
    return torch.cat(x + [torch.zeros(c.shape[0], 2, dtype=torch.float64, device=c.device)], 1)


def _forward64(w, x):
    h1 = torch.relu(x @ w[0].view(ENC, WIDTH) + w[1])
    h2 = torch.relu(h1 @ w[2].view(WIDTH, WIDTH) + w[3])
    h3 = torch.relu(h2 @ w[4].view(WIDTH, WIDTH) + w[5])
    return h3 @ w[6] + w[7]


def _infer64(case, seed):
    p, n = _surface_points(case["n"], seed)
    w = _model64(seed)
    return torch.cat([MU + SIGMA * _forward64(w, _encode64(a, b)) for a, b in zip(p.split(1 << 18), n.split(1 << 18))])


def _train64(case, seed):
    p, n = _surface_points(case["n"] * case["steps"], seed)
    t = _log_rho(p, n, seed).double()
    w = [v.requires_grad_(True) for v in _model64(seed)]
    m = [torch.zeros_like(v) for v in w]
    s = [torch.zeros_like(v) for v in w]
    for k in range(case["steps"]):
        a = slice(k * case["n"], (k + 1) * case["n"])
        y = _forward64(w, _encode64(p[a], n[a]))
        grad = torch.autograd.grad(torch.mean((y - (t[a] - MU) / SIGMA) ** 2), w)
        with torch.no_grad():
            for v, g, m1, s1 in zip(w, grad, m, s):
                m1.mul_(0.9).add_(g, alpha=0.1)
                s1.mul_(0.999).add_(g * g, alpha=0.001)
                mh, sh = m1 / (1 - 0.9 ** (k + 1)), s1 / (1 - 0.999 ** (k + 1))
                v -= 2e-3 * mh / (torch.sqrt(sh) + 1e-8)
    return torch.cat([v.detach().reshape(-1) for v in w]).cpu().numpy()


def _points64(case, seed):
    p, _ = _surface_points(case["n"], seed)
    q, _ = _surface_points(case["queries"], seed + 3)
    q[::2] = p[torch.arange(q[::2].shape[0], device=q.device) % p.shape[0]]
    radius = ctypes.c_float(case["radius"]).value
    pd, out = p.double(), []
    for a in q.double().split(max(1, (1 << 25) // case["n"])):
        d2 = sum((a[:, None, c] - pd[None, :, c]) ** 2 for c in range(3))
        m = (d2 < radius * radius).sum(1).double()
        rho = m / (math.pi * radius * radius)
        if case["density"] == "knn" and case["n"] >= case["k"]:
            dk2 = torch.topk(d2, case["k"], dim=1, largest=False).values[:, -1]
            rho = torch.where(m >= case["k"], case["k"] / (math.pi * dk2), rho)
        out.append(rho)
    return torch.cat(out)


def exact(case, seed):
    kind = case["kind"]
    if kind == "infer":
        return _infer64(case, seed)
    if kind == "train":
        return _train64(case, seed)
    if kind == "points" and float(case["n"]) * case["queries"] < 4.5e10:
        return _points64(case, seed)
    return None  # renders and the octree: no closed form
