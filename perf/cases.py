"""Performance cases of the library: what is timed, on which inputs, and what the outputs are
in 64 bits.

The cases are whole calls of the public entry points: renders from a 64x64 preview to a
1920x1080 frame of a 4096-leaf scene, in every weight type and with every sampling option a
program uses in earnest, the allocation-free render of a tile, a training step, an autograd
pass in float32 and a training step of the learned proposal.  The scenes, trees, MLP shapes,
cameras and sample budgets follow the repository's three synthetic workloads (64x64 with 8
leaves, 800x800 with 512, 1920x1080 with 4096); ``draw`` varies all of them, with odd sizes.

Inputs are made on the GPU from the seed alone.  ``exact`` is a float64 reference of its own:
tree, traversal, sampling, MLPs, compositing and the gradients by autograd in plain numpy and
torch.
"""
from __future__ import annotations

import heapq
import math

import numpy as np
import torch

import paper_2310_01881_amd as am

DEV = "cuda"
DTYPES = {"f32": am.AMNERF_F32, "bf16": am.AMNERF_BF16, "fp8": am.AMNERF_FP8, "fp8act": am.AMNERF_FP8_ACT}


# ---------------------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------------------
def _scene(size, **kw):
    """The scene and MLP settings of the three workloads."""
    base = {
        "small": dict(grid=32, blobs=20, depth=3, leaves=8, n_hidden=2, hidden=32, s_max=64),
        "frame": dict(grid=128, blobs=200, depth=12, leaves=512, n_hidden=4, hidden=64, s_max=128),
        "large": dict(grid=256, blobs=2000, depth=12, leaves=4096, n_hidden=4, hidden=64, s_max=192),
    }[size]
    return dict(base, scene=size, **kw)


def listed():
    return [
        # a thumbnail or a preview while a tree is being tuned: the smallest call, where launches count
        dict(name="thumb_f32", kind="render", dtype="f32", option="plain", width=64, height=64, **_scene("small")),
        # one tile of a served frame through the allocation-free entry point: ordinary small calls
        dict(name="tile_static_bf16", kind="static", dtype="bf16", option="plain", width=64, height=64, **_scene("frame")),
        # the headline frame, every sample of the plain sampler
        dict(name="frame_bf16", kind="render", dtype="bf16", option="plain", width=800, height=800, **_scene("frame")),
        # the same frame as a float32 reference render (training targets are made this way)
        dict(name="frame_f32", kind="render", dtype="f32", option="plain", width=800, height=800, **_scene("frame")),
        # the headline path: samples planned by the learned proposal
        dict(name="frame_bf16_prop", kind="render", dtype="bf16", option="prop", width=800, height=800, **_scene("frame")),
        # hierarchical sampling with node MLPs, on a ragged frame
        dict(name="frame_bf16_hs", kind="render", dtype="bf16", option="hs", width=641, height=477, **_scene("frame")),
        # a full HD frame of the 4096-leaf scene: e4m3 weights (several passes on the render lanes)
        dict(name="large_fp8", kind="render", dtype="fp8", option="plain", width=1920, height=1080, **_scene("large")),
        # ... with e4m3 weights and activations on the float8 matrix cores
        dict(name="large_fp8act", kind="render", dtype="fp8act", option="plain", width=1920, height=1080, **_scene("large")),
        # ... with empty space skipped
        dict(name="large_fp8_ess", kind="render", dtype="fp8", option="ess", width=1920, height=1080, **_scene("large")),
        # fitting the leaf MLPs: forward, backward, Adam and the repack of one batch
        dict(name="train_bf16", kind="train", dtype="bf16", option="plain", rays=262144, **_scene("frame")),
        # a float32 fit through autograd with colour, depth and opacity in the loss
        dict(name="fit_f32", kind="fit", dtype="f32", option="plain", rays=16384,
             **dict(_scene("frame"), leaves=64, hidden=32, s_max=64)),
        # one training step of the proposal
        dict(name="prop_train", kind="prop_train", dtype="bf16", option="plain", rays=32768, **_scene("frame")),
    ]


def draw(rng):
    """One more case: any of the kinds, sizes spread over their ranges."""
    def logint(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["render", "render", "render", "render", "static", "train", "fit", "prop_train"])
    size = rng.choice(["small", "frame", "frame", "frame", "large"])
    c = dict(kind=kind, **_scene(size))
    c["leaves"] = {"small": rng.randint(2, 8), "frame": logint(16, 1024), "large": logint(1024, 4096)}[size]
    c["s_max"] = rng.choice([24, 48, 64, 96, 128, 160, 192, 255])
    c["n_hidden"] = rng.choice([2, 3, 4, 4, 4])
    c["hidden"] = rng.choice([32, 64, 64])
    c["option"] = "plain"
    if kind == "render":
        c["dtype"] = rng.choice(["f32", "bf16", "bf16", "fp8", "fp8act"])
        c["option"] = rng.choice(["plain", "plain", "prop", "ess", "hs", "rounds"])
        if c["option"] == "hs":
            c["leaves"] = min(c["leaves"], 1024)
        if c["dtype"] != "fp8act" and c["option"] == "plain" and rng.random() < 0.3:
            c["n_hidden"] = rng.choice([1, 6, 8])
            if c["dtype"] == "f32":
                c["hidden"] = 32
        c["width"], c["height"] = logint(48, 800), logint(48, 640)
        if c["dtype"] == "f32":
            c["width"], c["height"] = min(c["width"], 500), min(c["height"], 500)
    elif kind == "static":
        c["dtype"] = rng.choice(["bf16", "bf16", "f32", "fp8"])
        c["s_max"] = rng.choice([32, 64, 96, 128])
        c["width"], c["height"] = logint(16, 80), logint(16, 80)
    elif kind == "train":
        c["dtype"] = rng.choice(["bf16", "bf16", "bf16", "f32"])
        c["rays"] = logint(2000, 200000 if c["dtype"] == "bf16" else 20000)
        c["leaves"] = min(c["leaves"], 1024)
    elif kind == "fit":
        c["dtype"] = rng.choice(["f32", "bf16"])
        c["rays"] = logint(1000, 40000)
        c["leaves"] = min(c["leaves"], 512)
    else:
        c["dtype"] = rng.choice(["bf16", "f32"])
        c["rays"] = logint(4000, 40000)
    if c["dtype"] == "fp8act":
        c["hidden"] = 64
    return c


def _n_rays(case):
    return case["rays"] if "rays" in case else case["width"] * case["height"]


def _flop_per_sample(case):
    h, n = case["hidden"], case["n_hidden"]
    return 2 * (30 * h + (n - 1) * h * h + 4 * h)


def _params(case):
    h, n = case["hidden"], case["n_hidden"]
    return 30 * h + h + (n - 1) * (h * h + h) + 4 * h + 4


def _samples(case):
    """Samples a pass evaluates: about three quarters of the budget where the scene fills the
    frame, fewer where options drop them (measured averages of the listed cases)."""
    part = {"prop": 0.22, "ess": 0.19, "hs": 0.29}.get(case["option"], 0.44 if case["scene"] == "large" else 0.75)
    return part * _n_rays(case) * case["s_max"]


def work(case):
    """Each ray read once (24 B), its colour, depth and opacity written once (20 B), every
    parameter read once; a training step also reads targets and reads and writes parameters and
    Adam moments.  The leaf MLPs' multiply-adds: once forward, and for a backward pass the input
    gradients and the weight gradients as well (the recomputed forward is not counted)."""
    R, ns, fl = _n_rays(case), _samples(case), _flop_per_sample(case)
    weight = {"f32": 4, "bf16": 2, "fp8": 1, "fp8act": 1}[case["dtype"]]
    sets = case["leaves"] * (2 if case["option"] == "hs" else 1)
    if case["kind"] in ("render", "static"):
        return {"bytes": 44.0 * R + sets * _params(case) * weight, "flops": ns * fl}
    if case["kind"] == "train":
        return {"bytes": 36.0 * R + sets * _params(case) * 32.0, "flops": 3 * ns * fl}
    if case["kind"] == "fit":
        return {"bytes": 64.0 * R + sets * _params(case) * 8.0, "flops": 3 * ns * fl}
    intervals = 0.1 * ns
    return {"bytes": 24.0 * R + sets * _params(case) * weight, "flops": ns * fl + 3 * intervals * 17792}


# ---------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------
def _gen(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed((seed * 1000003 + stream) % (1 << 62))
    return g


def _uniform(g, lo, hi, *shape):
    return lo + (hi - lo) * torch.rand(*shape, generator=g, device=DEV, dtype=torch.float64)


def _grid(case, seed):
    """Guidance densities: axis-aligned Gaussian blobs (separable, so their sum is one matrix
    product), a ground slab in the 800x800 scene, nine tenths of the blobs in one octant in the
    large one; rounded to 2^-10, float32[n^3], x fastest."""
    n, b = case["grid"], case["blobs"]
    g = _gen(seed, 1)
    lo, hi = {"small": (0.05, 0.2), "frame": (0.02, 0.15), "large": (0.01, 0.08)}[case["scene"]]
    mu = _uniform(g, 0.1, 0.9, b, 3)
    if case["scene"] == "large":
        mu = _uniform(g, 0.0, 1.0, b, 3)
        mu[: b * 93 // 100] *= 0.5
    s = _uniform(g, lo, hi, b, 3)
    amp = _uniform(g, 5.0, 50.0, b)
    c = (torch.arange(n, device=DEV, dtype=torch.float64) + 0.5) / n
    e = torch.exp(-0.5 * ((c[None, None, :] - mu[:, :, None]) / s[:, :, None]) ** 2)   # [b][3][n]
    zy = (e[:, 2, :, None] * e[:, 1, None, :]).reshape(b, n * n)
    out = (zy * amp[:, None]).T @ e[:, 0]                                              # [z y][x]
    out = torch.where(out < 1e-2, 0.0, out).reshape(n, n, n)
    if case["scene"] == "frame":
        out[:10] += 100.0
    return (torch.round(out * 1024.0) / 1024.0).float().reshape(-1)


def _camera_axes(g, n):
    """n cameras on a sphere of radius 2 around the scene centre, looking at it: position, forward,
    right and up vectors, each [n][3]."""
    u = torch.randn(n, 3, generator=g, device=DEV, dtype=torch.float64)
    u[:, 2] = u[:, 2].clamp(-1.5, 1.5)
    u[:, :2] += torch.where(u[:, :2] >= 0, 0.3, -0.3)
    u = u / u.norm(dim=1, keepdim=True)
    up = torch.zeros_like(u)
    up[:, 2] = 1.0
    r = torch.linalg.cross(-u, up)
    r = r / r.norm(dim=1, keepdim=True)
    return 0.5 + 2.0 * u, -u, r, torch.linalg.cross(r, -u)


def _rays(case, seed):
    """Rays through the pixel centres of one camera, or through random pixels of 100 cameras."""
    g = _gen(seed, 2)
    th = math.tan(math.radians(40.0) / 2.0)
    if "rays" in case:
        w = h = 800
        pos, f, r, u = _camera_axes(g, 100)
        cam = torch.randint(0, 100, (case["rays"],), generator=g, device=DEV)
        px = torch.randint(0, w * h, (case["rays"],), generator=g, device=DEV)
        pos, f, r, u = pos[cam], f[cam], r[cam], u[cam]
    else:
        w, h = case["width"], case["height"]
        pos, f, r, u = _camera_axes(g, 1)
        px = torch.arange(w * h, device=DEV)
        if case["kind"] == "static":      # a tile of an 800x800 frame around its centre
            px = (px // w + 400 - h // 2) * 800 + px % w + 400 - w // 2
            w = h = 800
        pos = pos.expand(px.numel(), 3)
    x = (((px % w) + 0.5) / w * 2.0 - 1.0) * th * (w / h)
    y = (1.0 - ((px // w) + 0.5) / h * 2.0) * th
    d = f + x[:, None] * r + y[:, None] * u
    d = d / d.norm(dim=1, keepdim=True)
    return pos.T.float().contiguous(), d.T.float().contiguous()


def _dims(case):
    h, n = case["hidden"], case["n_hidden"]
    return [(30, h)] + [(h, h)] * (n - 1) + [(h, 4)]


def _weights(case, seed, density):
    """He-normal parameters with zero biases, but the density output's, which is softplus^-1 of
    the node's mean guidance density."""
    g = _gen(seed, 3)
    parts = []
    n = density.numel()
    for fi, fo in _dims(case):
        parts.append(torch.randn(n, fi * fo, generator=g, device=DEV) * math.sqrt(2.0 / fi))
        parts.append(torch.zeros(n, fo, device=DEV))
    y = density.clamp_min(1e-4)
    parts[-1][:, 0] = torch.where(y > 30.0, y, torch.log(torch.expm1(y.clamp_max(30.0)))).float()
    return torch.cat(parts, 1).contiguous()


def _node_density(rows, mass, gmax):
    vol = np.prod((rows[:, 5:8] - rows[:, 2:5]).astype(np.float64), axis=1)
    return mass.astype(np.float64) * (gmax / 2.0 ** 24) / vol


def _set_density(case, rows, mass, gmax):
    """Mean guidance density of every parameter set's box, in slot order."""
    dens = _node_density(rows, mass, gmax)
    if case["option"] == "hs":
        return torch.from_numpy(dens[np.argsort(rows[:, 11])].copy()).to(DEV)
    leaf = rows[:, 10] >= 0
    return torch.from_numpy(dens[leaf][np.argsort(rows[leaf, 10])].copy()).to(DEV)


def _prop_features(o, d, t0, t1, k, s_max, centre, size):
    q = (o - 0.5) * 0.5
    f = [q, d]
    for v in (q, d):
        for fr in (math.pi, 2.0 * math.pi):
            f += [torch.sin(fr * v), torch.cos(fr * v)]
    f += [(k / s_max)[:, None], 2.0 * centre - 1.0, size, 2.0 * (o + t0[:, None] * d) - 1.0, 2.0 * (o + t1[:, None] * d) - 1.0]
    return torch.cat(f, 1)


def _prop_weights(case, seed, rows, density, o, d):
    """Proposal parameters: two layers of He-normal ReLU features and an output layer fitted by
    least squares to the optical thickness that the guidance density gives (4096 rays against
    random leaves), so that plans look like a trained network's; rounded to 2^-12."""
    g = _gen(seed, 4)
    w0 = torch.randn(64, 43, generator=g, device=DEV, dtype=torch.float64) * math.sqrt(2.0 / 43)
    w1 = torch.randn(64, 64, generator=g, device=DEV, dtype=torch.float64) * math.sqrt(2.0 / 64)
    leaf = rows[rows[:, 10] >= 0]
    leaf = torch.from_numpy(leaf[np.argsort(leaf[:, 10])].copy()).to(DEV).double()
    lo, hi = leaf[:, 2:5] / case["grid"], leaf[:, 5:8] / case["grid"]
    n = o.shape[1]
    pick = torch.randint(0, n, (4096,), generator=g, device=DEV)
    ro, rd = o[:, pick].T.double(), d[:, pick].T.double()
    box = torch.randint(0, lo.shape[0], (min(512, lo.shape[0]),), generator=g, device=DEV)
    a = (lo[box][None] - ro[:, None]) / rd[:, None]
    b = (hi[box][None] - ro[:, None]) / rd[:, None]
    t0 = torch.minimum(a, b).amax(2).clamp_min(0.0)
    t1 = torch.maximum(a, b).amin(2)
    ray, col = torch.nonzero(t1 > t0 + 1e-4, as_tuple=True)
    ray, col = ray[:60000], col[:60000]
    t0, t1, bx = t0[ray, col], t1[ray, col], box[col]
    k = torch.floor(12.0 * (t0 - 1.2) / 1.8).clamp(0, 30)
    f = _prop_features(ro[ray], rd[ray], t0, t1, k, case["s_max"], 0.5 * (lo[bx] + hi[bx]), hi[bx] - lo[bx])
    h = torch.relu(torch.relu(f @ w0.T) @ w1.T)
    tau = (density[bx] * (t1 - t0) / 32.0).clamp(1e-4, 8.0)
    y = torch.log(torch.expm1(tau))
    hb = torch.cat([h, torch.ones_like(h[:, :1])], 1)
    sol = torch.linalg.solve(hb.T @ hb + 1e-2 * h.shape[0] * torch.eye(65, device=DEV, dtype=torch.float64), hb.T @ y)
    ramp = torch.linspace(-0.05, 0.05, 32, device=DEV, dtype=torch.float64)
    z64 = torch.zeros(64, device=DEV, dtype=torch.float64)
    out = torch.cat([w0.reshape(-1), z64, w1.reshape(-1), z64, (sol[:64, None] * (1.0 + ramp)).T.reshape(-1), sol[64] + ramp])
    return (torch.round(out * 4096.0) / 4096.0).float().contiguous()


_CTX = []


def _context():
    """The one context that a program keeps."""
    if not _CTX:
        _CTX.append(am.Context(0))
    return _CTX[0]


def _targets(case, seed, d):
    """Colours of a smooth image over the view directions."""
    a = _uniform(_gen(seed, 5), -4.0, 4.0, 3, 4)
    return (0.5 + 0.45 * torch.sin(a[:, :3].float() @ d + a[:, 3:].float())).T.contiguous()


def prepare(case, seed):
    ctx = _context()
    grid = _grid(case, seed)
    host = grid.cpu().numpy()
    tree = am.Tree(ctx, host, case["grid"], case["depth"], case["leaves"])
    o, d = _rays(case, seed)
    gmax = float(host.max())
    density = _set_density(case, tree.rows, tree.mass, gmax)
    n_sets = density.numel()
    master = _weights(case, seed, density)
    st = {"case": case, "ctx": ctx, "tree": tree, "o": o, "d": d}
    dt = DTYPES[case["dtype"]]
    nh, h = case["n_hidden"], case["hidden"]
    if case["kind"] == "train":
        t = am.Trainer(ctx, tree, master, nh, h, f32=case["dtype"] == "f32")
        g = _gen(seed, 6)                # Adam's moments as in the middle of a fit
        t.m.copy_(torch.randn(t.m.shape, generator=g, device=DEV) * 1e-6)
        t.v.copy_((torch.rand(t.v.shape, generator=g, device=DEV) + 0.5) * 1e-10)
        t.step_no = 1000
        return dict(st, trainer=t, target=_targets(case, seed, d))
    if case["kind"] == "fit":
        R = case["rays"]
        return dict(st, master=master.requires_grad_(True), target=_targets(case, seed, d), R=R)
    if case["option"] == "hs":
        st["footprint"] = 0.25
    if dt == am.AMNERF_FP8_ACT:
        # activation scales from a calibration render of some of the pixels (two layers of the
        # same call a program makes once per scene)
        step = max(1, o.shape[1] // 65536)
        co, cd = o[:, ::step].contiguous(), d[:, ::step].contiguous()
        plain = am.Mlp(ctx, master, nh, h, am.AMNERF_BF16, n_sets)
        am.render(ctx, tree, plain, co, cd, case["s_max"], hcheck_footprint=st.get("footprint", 0.0))
        amax = torch.zeros((n_sets, nh), device=DEV)
        am.amnerf_mlp_calibrate(ctx.h, nh, n_sets, master, co, cd, amax)
        st["mlp"] = am.Mlp(ctx, master, nh, h, dt, n_sets, act_max_dev=amax)
    else:
        st["mlp"] = am.Mlp(ctx, master, nh, h, dt, n_sets)
    if case["option"] == "ess":
        st["occ"] = am.Occupancy(ctx, host, case["grid"], 2, 0.01)
    if case["option"] == "prop" or case["kind"] == "prop_train":
        p = am.Proposal(ctx, _prop_weights(case, seed, tree.rows, density, o, d))
        if case["kind"] == "prop_train":
            g = _gen(seed, 7)
            p.m.copy_(torch.randn(p.m.shape, generator=g, device=DEV) * 1e-5)
            p.v.copy_((torch.rand(p.v.shape, generator=g, device=DEV) + 0.5) * 1e-8)
            p.step_no = 500
        else:
            st["desc"] = p.descriptor(am.AMNERF_BF16, 0.95, min(48, case["s_max"]))
        st["prop"] = p
    if case["kind"] == "static":
        R = o.shape[1]
        st["out"] = [torch.empty((R, 3), device=DEV), torch.empty(R, device=DEV), torch.empty(R, device=DEV)]
    return st


def run(st):
    case, ctx, tree, o, d = st["case"], st["ctx"], st["tree"], st["o"], st["d"]
    s_max = case["s_max"]
    if case["kind"] == "train":
        t = st["trainer"]
        loss = t.step(o, d, st["target"], s_max)
        return {"loss": loss, "grad": t.grad, "master": t.master}
    if case["kind"] == "fit":
        m = st["master"]
        m.grad = None
        rgb, depth, opac = am.RenderFn.apply(m, ctx, tree, o, d, s_max, 1e-4, case["n_hidden"], case["hidden"],
                                             DTYPES[case["dtype"]])
        loss = ((rgb - st["target"]) ** 2).mean() + 0.1 * ((depth - 1.5) ** 2).mean() + 0.1 * ((opac - 1.0) ** 2).mean()
        loss.backward()
        return {"rgb": rgb.detach(), "depth": depth.detach(), "opacity": opac.detach(), "grad": m.grad}
    if case["kind"] == "prop_train":
        p = st["prop"]
        loss = p.train_step(tree, st["mlp"].desc, o, d, s_max)
        return {"loss": loss, "grad": p.grad, "master": p.master}
    if case["kind"] == "static":
        rgb, depth, opac = st["out"]
        am.amnerf_render_static(ctx.h, tree.h, st["mlp"].desc, o, d, s_max, rgb, depth, opac)
        return {"rgb": rgb, "depth": depth, "opacity": opac}
    if case["option"] == "rounds":
        R = o.shape[1]
        rgb, depth, opac = torch.empty((R, 3), device=DEV), torch.empty(R, device=DEV), torch.empty(R, device=DEV)
        am.amnerf_render(ctx.h, tree.h, st["mlp"].desc, o, d, s_max, rgb, depth, opac, ert_rounds=True)
        return {"rgb": rgb, "depth": depth, "opacity": opac}
    return am.render(ctx, tree, st["mlp"], o, d, s_max, hcheck_footprint=st.get("footprint", 0.0),
                     occupancy=st.get("occ"), proposal=st.get("desc"))


# ---------------------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------------------
def _quantised(host):
    g = np.maximum(host.astype(np.float64), 0.0)
    return np.floor(np.ldexp(g / g.max(), 24) + 0.5).astype(np.int64)


def _ref_tree(case, host):
    """Best-first density-median tree: rows as the library exports them, and the node list
    (lo, hi, axis, plane, left) with the root first."""
    n = case["grid"]
    s = np.zeros((n + 1, n + 1, n + 1), np.int64)
    s[1:, 1:, 1:] = _quantised(host).reshape(n, n, n).cumsum(0).cumsum(1).cumsum(2)

    def box(lo, hi):
        v = 0
        for k, sk in ((hi[2], 1), (lo[2], -1)):
            for j, sj in ((hi[1], 1), (lo[1], -1)):
                v += sk * sj * (int(s[k, j, hi[0]]) - int(s[k, j, lo[0]]))
        return v

    nodes = [dict(lo=[0, 0, 0], hi=[n, n, n], code=1, depth=0, mass=box([0, 0, 0], [n, n, n]), left=-1, axis=-1, plane=-1)]
    heap = []

    def offer(i):
        nd = nodes[i]
        ext = [nd["hi"][a] - nd["lo"][a] for a in range(3)]
        nd["a"] = max(range(3), key=lambda a: (ext[a], -a))
        if nd["depth"] < case["depth"] and max(ext) >= 2:
            heapq.heappush(heap, (-nd["mass"], nd["code"], i))

    offer(0)
    leaves = 1
    while heap and leaves < case["leaves"]:
        _, _, i = heapq.heappop(heap)
        nd = nodes[i]
        a, lo, hi = nd["a"], nd["lo"], nd["hi"]
        if nd["mass"] == 0:
            plane = (lo[a] + hi[a]) // 2
        else:
            L, R, plane = lo[a] + 1, hi[a] - 1, hi[a] - 1
            while L <= R:
                mid = (L + R) // 2
                if 2 * box(lo, [mid if x == a else hi[x] for x in range(3)]) >= nd["mass"]:
                    plane, R = mid, mid - 1
                else:
                    L = mid + 1
        nd.update(axis=a, plane=plane, left=len(nodes))
        lhi = [plane if x == a else hi[x] for x in range(3)]
        rlo = [plane if x == a else lo[x] for x in range(3)]
        lm = box(lo, lhi)
        for q, (l2, h2, m2) in enumerate(((lo, lhi, lm), (rlo, hi, nd["mass"] - lm))):
            nodes.append(dict(lo=list(l2), hi=list(h2), code=2 * nd["code"] + q, depth=nd["depth"] + 1, mass=m2, left=-1,
                              axis=-1, plane=-1))
            offer(len(nodes) - 1)
        leaves += 1
    stack, slot, nslot = [0], 0, 0
    while stack:
        nd = nodes[stack.pop()]
        nd["nslot"], nslot = nslot, nslot + 1
        nd["slot"] = -1
        if nd["left"] < 0:
            nd["slot"], slot = slot, slot + 1
        else:
            stack += [nd["left"] + 1, nd["left"]]
    order = sorted(range(len(nodes)), key=lambda i: nodes[i]["code"])
    rows = np.array([[nodes[i]["code"], nodes[i]["depth"], *nodes[i]["lo"], *nodes[i]["hi"], nodes[i]["axis"], nodes[i]["plane"],
                      nodes[i]["slot"], nodes[i]["nslot"]] for i in order], np.int64)
    return nodes, rows, np.array([nodes[i]["mass"] for i in order], np.uint64)


def _ref_intervals(case, nodes, o, d, footprint):
    """Intervals of every ray, ray-major and front to back: ray, t0, t1, parameter set, samples."""
    n, R = case["grid"], o.shape[0]
    inf = torch.full((R,), math.inf, device=DEV, dtype=torch.float64)
    t0, t1 = torch.zeros_like(inf), inf.clone()
    ok = torch.ones(R, dtype=torch.bool, device=DEV)
    for a in range(3):
        flat = d[:, a] == 0
        ta, tb = (0.0 - o[:, a]) / d[:, a], (1.0 - o[:, a]) / d[:, a]
        t0 = torch.where(flat, t0, torch.maximum(t0, torch.minimum(ta, tb)))
        t1 = torch.where(flat, t1, torch.minimum(t1, torch.maximum(ta, tb)))
        ok &= ~(flat & ((o[:, a] < 0) | (o[:, a] > 1)))
    ids = torch.nonzero(ok & (t0 < t1)).reshape(-1)
    stack = [(0, ids, t0[ids], t1[ids], torch.zeros(ids.numel(), dtype=torch.bool, device=DEV))]
    m = torch.zeros(R, dtype=torch.int64, device=DEV)
    found = []
    while stack:
        i, r, a0, a1, gone = stack.pop()     # gone: a node above took the ray's segment
        if not r.numel():
            continue
        nd = nodes[i]
        leaf = nd["left"] < 0
        take = ~gone
        if leaf:
            m[r] += 1
        elif footprint > 0:
            side = np.float32(max(nd["hi"][x] - nd["lo"][x] for x in range(3)) / n)
            take = take & (a0.float() > float(side / np.float32(footprint)))
        else:
            take = torch.zeros_like(gone)
        if bool(take.any()):
            found.append((r[take], a0[take], a1[take], torch.full_like(r[take], nd["slot"] if footprint <= 0 else nd["nslot"])))
        if leaf:
            continue
        gone = gone | take
        ax, s = nd["axis"], nd["plane"] / n
        oa, da = o[r, ax], d[r, ax]
        upper_first = torch.where(da == 0, oa >= s, da < 0)
        ts = torch.where(da == 0, torch.full_like(da, math.inf), (s - oa) / da)
        only_before, only_after = ts >= a1, (ts <= a0) & ~(ts >= a1)
        for child in (1, 0):
            first = upper_first == bool(child)
            on = torch.where(first, ~only_after, ~only_before)
            c0 = torch.where(first | only_after, a0, ts)
            c1 = torch.where(first & ~only_before, ts, a1)
            stack.append((nd["left"] + child, r[on], c0[on], c1[on], gone[on]))
    ray, u0, u1, key = (torch.cat(x) for x in zip(*found))
    by = torch.argsort(u0, stable=True)
    by = by[torch.argsort(ray[by], stable=True)]
    ray, u0, u1, key = ray[by], u0[by], u1[by], key[by]
    first = torch.searchsorted(ray, torch.arange(R, device=DEV))
    k = torch.arange(ray.numel(), device=DEV) - first[ray]
    S = case["s_max"]
    npi = torch.where(m <= S, S // m.clamp_min(1), 1)
    keep = k < S
    return ray[keep], u0[keep], u1[keep], key[keep], npi[ray[keep]], k[keep]


def _ref_mlp(case, master, key, p, d):
    """Pre-activations of the samples (sample order kept): every parameter set over its samples."""
    x = 2.0 * p - 1.0
    f = [x]
    for q in range(4):
        f += [torch.sin(math.pi * 2.0 ** q * x), torch.cos(math.pi * 2.0 ** q * x)]
    f = torch.cat(f + [d], 1)
    order = torch.argsort(key, stable=True)
    f = f[order]
    n_sets = master.shape[0]
    count = torch.bincount(key, minlength=n_sets).tolist()
    out, at = [], 0
    sets = master.unbind(0)
    dims = _dims(case)
    for b, c in enumerate(count):
        if not c:
            continue
        h, off = f[at:at + c], 0
        at += c
        for layer, (fi, fo) in enumerate(dims):
            w = sets[b][off:off + fi * fo].view(fo, fi)
            h = torch.addmm(sets[b][off + fi * fo:off + fi * fo + fo], h, w.T)
            off += fi * fo + fo
            if layer + 1 < len(dims):
                h = torch.relu(h)
        out.append(h)
    z = torch.cat(out) if out else f.new_zeros(0, 4)
    back = torch.empty_like(order)
    back[order] = torch.arange(order.numel(), device=DEV)
    return z[back]


def _softplus(z):
    return z.clamp_min(0) + torch.log1p(torch.exp(-z.abs()))


def _ref_render(case, nodes, master, o, d, footprint=0.0, occ=None, eps=1e-4):
    """rgb, depth, opacity, the intervals and the samples' densities."""
    R, S = o.shape[0], case["s_max"]
    iv = _ref_intervals(case, nodes, o, d, footprint)
    ray, t0, t1, key, npi, _ = iv
    which = torch.repeat_interleave(torch.arange(ray.numel(), device=DEV), npi)
    first = torch.cumsum(npi, 0) - npi
    j = torch.arange(which.numel(), device=DEV) - first[which]
    delta = ((t1 - t0) / npi)[which]
    t = t0[which] + (j + 0.5) * delta
    rs = ray[which]
    p = o[rs] + t[:, None] * d[rs]
    z = _ref_mlp(case, master, key[which], p, d[rs])
    sigma = _softplus(z[:, 0])
    if occ is not None:
        g, cells = occ
        c = torch.floor(p * g).clamp(0, g - 1).long()
        sigma = torch.where(cells[c[:, 0] + g * (c[:, 1] + g * c[:, 2])], sigma, 0.0)
    colour = torch.sigmoid(z[:, 1:])
    head = torch.searchsorted(rs, torch.arange(R, device=DEV))
    slot = rs * S + (torch.arange(rs.numel(), device=DEV) - head[rs])
    tau = torch.zeros(R * S, device=DEV, dtype=torch.float64).index_put((slot,), sigma * delta).view(R, S)
    tt = torch.zeros(R * S, device=DEV, dtype=torch.float64).index_put((slot,), t).view(R, S)
    cc = torch.zeros(R * S, 3, device=DEV, dtype=torch.float64).index_put((slot,), colour).view(R, S, 3)
    run_sum = torch.cumsum(tau, 1)
    w = torch.exp(-(run_sum - tau)) * -torch.expm1(-tau)
    stop = torch.exp(-run_sum) < eps
    w = torch.where((torch.cumsum(stop.long(), 1) - stop.long()) > 0, 0.0, w)
    return (w[:, :, None] * cc).sum(1), (w * tt).sum(1), w.sum(1), iv, sigma


def _ref_adam(p, m, v, g, lr, step):
    m = 0.9 * m + (1.0 - 0.9) * g
    v = 0.999 * v + (1.0 - 0.999) * g * g
    return p - lr * (m / (1.0 - 0.9 ** step)) / ((v / (1.0 - 0.999 ** step)).sqrt() + 1e-8)


def exact(case, seed):
    # the plan of a proposal is a discrete choice that the bfloat16 network takes: no value in
    # 64 bits; and no more than some seconds of float64 products
    times = 1 if case["kind"] in ("render", "static", "prop_train") else 3
    if case["option"] == "prop" or times * 0.9 * _n_rays(case) * case["s_max"] * _flop_per_sample(case) > 1.5e14:
        return None
    host = _grid(case, seed).cpu().numpy()
    nodes, rows, mass = _ref_tree(case, host)
    o32, d32 = _rays(case, seed)
    o, d = o32.T.double(), d32.T.double()
    density = _set_density(case, rows, mass, float(host.max()))
    master = _weights(case, seed, density).double()
    R = o.shape[0]
    if case["kind"] in ("render", "static"):
        occ = None
        if case["option"] == "ess":
            g = case["grid"] // 2
            q = torch.from_numpy(_quantised(host)).to(DEV).view(g, 2, g, 2, g, 2).amax((1, 3, 5))
            occ = (g, (q >= max(1, math.floor(float(np.float32(0.01)) * 2.0 ** 24 + 0.5))).reshape(-1))
        rgb, depth, opac, _, _ = _ref_render(case, nodes, master, o, d, 0.25 if case["option"] == "hs" else 0.0, occ)
        return {"rgb": rgb, "depth": depth, "opacity": opac}
    target = _targets(case, seed, d32).double()
    if case["kind"] in ("train", "fit"):
        master.requires_grad_(True)
        rgb, depth, opac, _, _ = _ref_render(case, nodes, master, o, d)
        loss = ((rgb - target) ** 2).mean()
        if case["kind"] == "fit":
            total = loss + 0.1 * ((depth - 1.5) ** 2).mean() + 0.1 * ((opac - 1.0) ** 2).mean()
            (grad,) = torch.autograd.grad(total, master)
            return {"rgb": rgb.detach(), "depth": depth.detach(), "opacity": opac.detach(), "grad": grad}
        (grad,) = torch.autograd.grad(loss, master)
        g = _gen(seed, 6)
        m = (torch.randn(master.shape, generator=g, device=DEV) * 1e-6).double()
        v = ((torch.rand(master.shape, generator=g, device=DEV) + 0.5) * 1e-10).double()
        return {"loss": loss.detach().view(1), "grad": grad, "master": _ref_adam(master.detach(), m, v, grad, 1e-3, 1001)}
    # the proposal's training step: targets from the plain render's densities
    _, _, _, (ray, t0, t1, key, npi, k), sigma = _ref_render(case, nodes, master, o, d, eps=0.0)
    which = torch.repeat_interleave(torch.arange(ray.numel(), device=DEV), npi)
    first = torch.cumsum(npi, 0) - npi
    j = (torch.arange(which.numel(), device=DEV) - first[which]).double()
    n = npi[which].double()
    tau = torch.zeros(ray.numel(), 32, device=DEV, dtype=torch.float64)
    for b in range(32):
        over = (torch.minimum((j + 1) / n, torch.full_like(j, (b + 1) / 32)) - torch.maximum(j / n, torch.full_like(j, b / 32)))
        tau[:, b].index_add_(0, which, sigma * (t1 - t0)[which] * over.clamp_min(0.0))
    want = -torch.expm1(-tau)
    leaf = rows[rows[:, 10] >= 0]
    leaf = torch.from_numpy(leaf[np.argsort(leaf[:, 10])].copy()).to(DEV).double()
    lo, hi = leaf[:, 2:5] / case["grid"], leaf[:, 5:8] / case["grid"]
    f = _prop_features(o[ray], d[ray], t0, t1, k.double(), case["s_max"], 0.5 * (lo + hi)[key], (hi - lo)[key])
    w = _prop_weights(case, seed, rows, density, o32, d32).double().requires_grad_(True)
    a, b = 64 * 43, 64 * 64
    h = torch.relu(f @ w[:a].view(64, 43).T + w[a:a + 64])
    h = torch.relu(h @ w[a + 64:a + 64 + b].view(64, 64).T + w[a + 64 + b:a + 128 + b])
    z = h @ w[a + 128 + b:a + 128 + b + 2048].view(32, 64).T + w[a + 128 + b + 2048:]
    loss = ((-torch.expm1(-_softplus(z)) - want) ** 2).mean()
    (grad,) = torch.autograd.grad(loss, w)
    g = _gen(seed, 7)
    m = (torch.randn(w.shape, generator=g, device=DEV) * 1e-5).double()
    v = ((torch.rand(w.shape, generator=g, device=DEV) + 0.5) * 1e-8).double()
    return {"loss": loss.detach().view(1), "grad": grad, "master": _ref_adam(w.detach(), m, v, grad, 1e-3, 501)}
