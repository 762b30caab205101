"""The places where a call takes another kernel, block size, tile or source of rows: the results
on both sides of each line, and the smallest, ragged and largest sizes of each."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import synth
from scene_util import Scene, gpu_setup, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2310_01881_amd as am  # noqa: E402
import test_gpu_ert as ert  # noqa: E402
import test_gpu_proposal as proposal  # noqa: E402
from test_gpu_render import check_intervals_and_sort, fetch_inspect, render_all  # noqa: E402


def small_scene(**kw):
    return Scene(synth.scaled(synth.C1, **kw))


@pytest.mark.parametrize("dtype", [am.AMNERF_F32, am.AMNERF_BF16])
def test_a_ray_does_not_depend_on_the_size_of_its_launch(dtype):
    """Blocks of one wave below 65 536 rays, of four from there on; chained scans, sort and rows
    from one ray to several tiles.  Every ray bit-equal to itself in the largest launch."""
    scene = small_scene(s_max=33)
    ctx, tree, mlp = gpu_setup(scene, dtype)
    o, d = synth.random_rays(65537, 3)

    def run(n):
        out = render_all(scene, ctx, tree, mlp, o[:, :n], d[:, :n], 33)
        _, ins = fetch_inspect(ctx, n, scene.n_sets)
        return out, ins

    ref, ri = run(65537)
    ref = {k: ref[k].clone() for k in ("rgb", "depth", "opacity")}
    for n in (1, 63, 64, 65, 2047, 2049, 65535, 65536):
        print("rays", n, flush=True)
        out, ins = run(n)
        for k in ref:
            assert torch.equal(out[k], ref[k][:n]), (n, k)
        ni, ns = ins["ray_iv_off"][n], ins["ray_smp_off"][n]
        for k, m in (("ray_iv_off", n + 1), ("ray_smp_off", n + 1), ("ray_used", n), ("iv_t0", ni), ("iv_dt", ni),
                     ("iv_slot", ni), ("iv_n", ni), ("sample_out", ns)):
            assert np.array_equal(ins[k][:m], ri[k][:m]), (n, k)


def test_direction_components_without_a_reciprocal():
    """A component below 2^-126 takes the dividing crossings.  At 1e-38 the crossings are still
    finite (below about 6e-39 they are not, which the traversal has never handled): the intervals
    are those of a component of zero, as the ray moves less than 1e-37 along it, and the
    crossings of the other planes within 1e-6."""
    scene = small_scene(s_max=33)
    ctx, tree, mlp = gpu_setup(scene, am.AMNERF_F32)
    o, d = synth.random_rays(600, 4)
    for r in range(0, 600, 3):
        d[r % 9 // 3, r] = 0.0
    tiny = d.copy()
    for r in range(0, 600, 3):
        tiny[r % 9 // 3, r] = np.float32(1e-38) * (1 if r % 2 else -1)
    got = []
    for dd in (d, tiny):
        render_all(scene, ctx, tree, mlp, o, dd, 33)
        got.append(fetch_inspect(ctx, 600, scene.n_sets)[1])
    a, b = got
    for k in ("ray_iv_off", "iv_slot", "iv_n"):
        assert np.array_equal(a[k], b[k]), k
    for k in ("iv_t0", "iv_dt"):
        np.testing.assert_allclose(a[k], b[k], rtol=0, atol=1e-6)


@pytest.mark.parametrize("dtype,kw,n_rays,s_max", [
    (am.AMNERF_F32, {}, 1, 255),
    (am.AMNERF_F32, {}, 4095, 128),                                  # 2^19 - 128 flags: the scan's small tiles
    (am.AMNERF_BF16, dict(n_hidden=4, hidden=64), 4096, 128),        # 2^19: large tiles, none ragged
    (am.AMNERF_BF16, {}, 4097, 128),                                 # one more, ragged
    (am.AMNERF_FP8, {}, 65, 8),                                      # one sample per interval
    (am.AMNERF_FP8_ACT, dict(n_hidden=4, hidden=64), 300, 96),
])
def test_rows_from_intervals_equal_rows_from_records(dtype, kw, n_rays, s_max):
    """A single pass reads the sorted intervals, a pass in rounds the compacted sample records:
    bit-equal outputs, weights and stop indices."""
    scene = small_scene(**kw)
    ctx, tree, mlp = gpu_setup(scene, dtype)
    o, d = (to_dev(a) for a in synth.random_rays(n_rays, 5))
    one, _, used1, off1 = ert.render(ctx, tree, mlp, o, d, s_max, 0, weights=True)
    two, _, used2, off2 = ert.render(ctx, tree, mlp, o, d, s_max, am.AMNERF_ERT_ROUNDS, weights=True)
    assert off1[-1] > 0
    ert.compare(two, one, (dtype, n_rays, s_max))
    assert np.array_equal(used1, used2) and np.array_equal(off1, off2)


@pytest.mark.parametrize("max_leaves,n_rays", [(1023, 300), (1500, 300), (1500, 9000)])
def test_sort_with_many_leaves(max_leaves, n_rays):
    """Above 1024 leaves a block is one wave, and segments are longer from 2^18 intervals on: the
    permutation and the buckets against the oracle."""
    scene = Scene(synth.scaled(synth.C2, grid_n=64, max_leaves=max_leaves, max_depth=12, n_hidden=1, hidden=32))
    assert scene.n_sets > 1000
    ctx, tree, mlp = gpu_setup(scene, am.AMNERF_BF16)
    o, d = synth.random_rays(n_rays, 6)
    render_all(scene, ctx, tree, mlp, o, d, 33)
    _, ins = fetch_inspect(ctx, n_rays, scene.n_sets)
    check_intervals_and_sort(scene, o, d, 33, ins, np.arange(0, n_rays, 31))


def test_compositing_more_than_64_intervals():
    """Rays of more than 64 intervals (the ones past those staged on chip are read from memory),
    as plain and as planned intervals, against float64 sums of the kernel's own samples.  Bar:
    a term's relative error is below 16 ulp (exponent up to 9.2, 1-ulp exponential, logarithm
    and reciprocal, a product of three), the terms sum to at most 1, and the sums round at most
    once per level of 64 and per window: 16 + 8 + 4 ulp of 2^-24, twice."""
    cfg = synth.scaled(synth.C2, grid_n=128, max_leaves=1500, max_depth=16, n_hidden=1, hidden=32, s_max=255)
    grid = np.zeros((128, 128, 128), np.float32)
    grid[:, 64, 64] = 3.0                                          # a line of voxels, and rays along it
    scene = Scene(cfg, grid=grid)
    ctx, tree, mlp = gpu_setup(scene, am.AMNERF_F32)
    prop = am.Proposal(ctx, torch.from_numpy(synth.make_prop_weights(1)).to("cuda:0"))
    rng = np.random.default_rng(7)
    o = (64.5 + rng.uniform(-0.3, 0.3, (3, 400))) / 128
    o[2] = -0.3
    d = rng.uniform(-1e-3, 1e-3, (3, 400))
    d[2] = 1.0
    o, d = o.astype(np.float32), (d / np.linalg.norm(d, axis=0, keepdims=True)).astype(np.float32)
    out = render_all(scene, ctx, tree, mlp, o, d, 255)
    _, ins = fetch_inspect(ctx, 400, scene.n_sets)
    m = np.diff(ins["ray_iv_off"].astype(np.int64))
    print("intervals per ray: up to", m.max())
    assert m.max() > 64 and ins["ray_used"].max() > 64
    rgb, op = out["rgb"].cpu().numpy(), out["opacity"].cpu().numpy()
    off, so = ins["ray_iv_off"].astype(np.int64), ins["ray_smp_off"].astype(np.int64)
    for r in range(400):
        u = int(ins["ray_used"][r])
        n = ins["iv_n"][off[r]:off[r + 1]]
        delta = np.repeat(ins["iv_dt"][off[r]:off[r + 1]] / n.astype(np.float32), n).astype(np.float64)[:u]
        z = ins["sample_out"][so[r]:so[r] + u].astype(np.float64)
        tau = np.logaddexp(0.0, z[:, 0]) * delta
        w = np.exp(-(np.cumsum(tau) - tau)) * -np.expm1(-tau)
        c = 1.0 / (1.0 + np.exp(-z[:, 1:]))
        assert abs(w.sum() - op[r]) <= 56 * 2.0 ** -24, r
        assert np.abs(w @ c - rgb[r]).max() <= 56 * 2.0 ** -24, r
    plain = proposal.render(ctx, tree, mlp, o, d, 255)
    planned = proposal.render(ctx, tree, mlp, o, d, 255, proposal=prop.descriptor(am.AMNERF_F32, mass_thresh=2.0, cap=255))
    for a, b in zip(plain[:3], planned[:3]):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("max_leaves,s_max", [(8, 1), (8, 33), (2, 64), (2, 255)])
def test_proposal_gradient_by_samples_per_interval(max_leaves, s_max):
    """Targets of intervals of 1 to 255 samples (half a wave takes 32 at a time).  The bars are
    those of the gradient test at the usual sample count."""
    cfg = synth.scaled(synth.C1, max_leaves=max_leaves, s_max=s_max)
    scene, ctx, tree, mlp, prop, prop_w = proposal.setup(cfg)
    o, d = synth.camera_rays(synth.make_cameras(1, cfg.seed_cameras, 9, 7)[0])
    loss = prop.train_step(tree, mlp.desc, to_dev(o), to_dev(d), s_max, lr=0.0).item()
    g = prop.grad.cpu().numpy().astype(np.float64)
    feat, _ = oracle.prop_eval(scene.otree, prop_w, o, d, s_max)
    alpha = oracle.prop_targets(scene.otree, scene.W, cfg.n_hidden, cfg.hidden, o, d, s_max)
    loss_ref, g_ref = oracle.prop_loss_grad(prop_w, feat, alpha)
    assert abs(loss - loss_ref) <= 1e-4 * loss_ref
    assert np.linalg.norm(g - g_ref) <= 1e-3 * np.linalg.norm(g_ref)


def sure_weights(n_sets, n_hidden, hidden, rng):
    """Weights whose hidden units are far from zero, half of them on and half off, whatever the
    input (|x| <= 1): the products are below 0.5 of the largest input, which stays below 6, and
    the biases are +-3.  No rounding can then switch a unit."""
    parts = []
    for l, (fi, fo) in enumerate(synth.layer_dims(n_hidden, hidden)):
        w = rng.uniform(-0.5 / fi, 0.5 / fi, (n_sets, fo, fi))
        b = np.where(rng.random((n_sets, fo)) < 0.5, 3.0, -3.0) if l < n_hidden else rng.uniform(-1, 1, (n_sets, fo))
        parts += [w.reshape(n_sets, -1), b]
    return np.concatenate(parts, axis=1).astype(np.float32)


def reference_gradient(scene, W, ins, gs, o, d, rnd):
    """Gradient of the leaf MLPs from the gradient `gs` at their outputs, in float64, with `rnd`
    where the kernel rounds its operands (weights, inputs, activations, gradients)."""
    n_hidden, hidden = scene.cfg.n_hidden, scene.cfg.hidden
    n = ins["iv_n"]
    which = np.repeat(np.arange(len(n)), n)
    j = np.arange(len(which)) - np.repeat(np.cumsum(n) - n, n)
    ray = np.repeat(np.arange(o.shape[1]), np.diff(ins["ray_iv_off"]))[which]
    delta = (ins["iv_dt"] / n.astype(np.float32))[which].astype(np.float64)
    t = ((j + 0.5) * delta + ins["iv_t0"][which].astype(np.float64)).astype(np.float32).astype(np.float64)
    dr, orr = d.T[ray].astype(np.float64), o.T[ray].astype(np.float64)
    p = (2.0 * (t[:, None] * dr + orr).astype(np.float32).astype(np.float64) - 1.0).astype(np.float32).astype(np.float64)
    f = [p]
    for k in range(4):
        f += [np.sin(np.pi * 2.0 ** k * p), np.cos(np.pi * 2.0 ** k * p)]
    x = rnd(np.concatenate(f + [dr], axis=1))
    slot = ins["iv_slot"][which]
    g = np.zeros(W.shape)
    dims = list(synth.layer_dims(n_hidden, hidden))
    offs = np.cumsum([0] + [fi * fo + fo for fi, fo in dims])
    for s in np.unique(slot):
        w = [rnd(W[s, a:a + fi * fo].astype(np.float64)).reshape(fo, fi) for a, (fi, fo) in zip(offs, dims)]
        h = [x[slot == s]]
        for l, (fi, fo) in enumerate(dims[:-1]):
            b = W[s, offs[l] + fi * fo:offs[l] + fi * fo + fo].astype(np.float64)
            h.append(rnd(np.maximum(h[-1] @ w[l].T + b, 0.0)))
        dz = rnd(gs[slot == s].astype(np.float64))
        for l in range(len(dims) - 1, -1, -1):
            fi, fo = dims[l]
            g[s, offs[l]:offs[l] + fi * fo] = (dz.T @ h[l]).ravel()
            g[s, offs[l] + fi * fo:offs[l] + fi * fo + fo] = dz.sum(axis=0)
            if l:
                dz = rnd((dz @ w[l]) * (h[l] > 0.0))
    return g


@pytest.mark.parametrize("dtype,n_hidden,hidden,n_rays,cap", [
    (am.AMNERF_BF16, 1, 32, 1, 0), (am.AMNERF_BF16, 4, 32, 40, 0), (am.AMNERF_BF16, 1, 64, 40, 0),
    (am.AMNERF_BF16, 2, 64, 700, 0), (am.AMNERF_BF16, 3, 64, 1, 0), (am.AMNERF_BF16, 4, 64, 700, 0),
    (am.AMNERF_F32, 4, 32, 1, 0), (am.AMNERF_F32, 2, 64, 700, 0), (am.AMNERF_F32, 4, 32, 9000, 0),
    (am.AMNERF_F32, 4, 32, 9000, 4 << 30),                          # the longest segments
])
def test_mlp_backward_by_shape(dtype, n_hidden, hidden, n_rays, cap):
    """The leaf MLPs' backward over shapes and bucket sizes from a few rows to many tiles, and
    both segment lengths in float32.  Bars (relative L2 of the whole gradient): in float32,
    features and sums within a few 1e-6 (random rounding over up to 2e5 samples), 2e-5; in
    bfloat16, operands that round to the other neighbour (2^-8 apart) where the kernel's float32
    value differs in its last bits: about 1e-5 of a feature's size against a spacing of 4e-3, a
    share of 2e-3 at most, so 2^-8 sqrt(2e-3) = 2e-4, times a few layers: 2e-3."""
    scene = small_scene(n_hidden=n_hidden, hidden=hidden, s_max=33)
    W = sure_weights(scene.n_sets, n_hidden, hidden, np.random.default_rng(8))
    ctx = am.Context(0, cap)
    tree = am.Tree(ctx, scene.grid, scene.cfg.grid_n, scene.cfg.max_depth, scene.cfg.max_leaves)
    master = torch.from_numpy(W).to("cuda:0")
    mlp = am.Mlp(ctx, master, n_hidden, hidden, dtype, scene.n_sets)
    o, d = synth.random_rays(n_rays, 12)
    od, dd = to_dev(o), to_dev(d)
    rgb = torch.empty((n_rays, 3), device="cuda:0")
    am.amnerf_render(ctx.h, tree.h, mlp.desc, od, dd, 33, rgb, None, None, None, 0.0)
    grad = torch.empty_like(master)
    rng = np.random.default_rng(9)
    am.amnerf_render_backward(ctx.h, tree.h, mlp.desc, od, dd, to_dev(rng.standard_normal((n_rays, 3)).astype(np.float32)),
                              grad, None, None)
    _, ins = fetch_inspect(ctx, n_rays, scene.n_sets)
    ns = int(ins["ray_smp_off"][n_rays])
    assert ns > 0
    gs = torch.empty((ns, 4), device="cuda:0")
    am.amnerf_render_backward_inspect(ctx.h, gs)
    torch.cuda.synchronize()

    def rnd(a):
        t = torch.from_numpy(np.ascontiguousarray(a)).to(torch.float32)
        return (t if dtype == am.AMNERF_F32 else t.to(torch.bfloat16)).to(torch.float64).numpy()

    ref = reference_gradient(scene, W, ins, gs.cpu().numpy(), o, d, rnd)
    e = np.linalg.norm(grad.cpu().numpy().astype(np.float64) - ref) / np.linalg.norm(ref)
    print("dtype %d %dx%d, %d samples: relative L2 %.2e" % (dtype, n_hidden, hidden, ns, e), flush=True)
    assert e <= (2e-5 if dtype == am.AMNERF_F32 else 2e-3)


@pytest.mark.parametrize("n_hidden,hidden", [(2, 32), (4, 64)])
def test_float32_training_step_forward(n_hidden, hidden):
    """A float32 training step's forward runs on the float32 matrix instructions, a render's on
    split bfloat16 values: loss and gradient of both.  Bar: outputs differ by 1e-5 of their size
    at most (the bar of the per-sample test), which a squared error's gradient carries on at its
    own size, to the compositing's and the products': 5e-5."""
    scene = small_scene(n_hidden=n_hidden, hidden=hidden, s_max=33)
    W = sure_weights(scene.n_sets, n_hidden, hidden, np.random.default_rng(10))
    ctx = am.Context(0)
    tree = am.Tree(ctx, scene.grid, scene.cfg.grid_n, scene.cfg.max_depth, scene.cfg.max_leaves)
    o, d = (to_dev(a) for a in synth.random_rays(500, 13))
    target = to_dev(np.random.default_rng(1).uniform(0, 1, (500, 3)).astype(np.float32))
    tr = am.Trainer(ctx, tree, to_dev(W), n_hidden, hidden, f32=True)
    loss = tr.step(o, d, target, 33, grad_only=True).item()
    master = to_dev(W).requires_grad_(True)
    rgb, _, _ = am.RenderFn.apply(master, ctx, tree, o, d, 33, 1e-4, n_hidden, hidden, am.AMNERF_F32)
    l2 = ((rgb - target) ** 2).mean()
    l2.backward()
    e = ((master.grad - tr.grad).norm() / tr.grad.norm()).item()
    print("%dx%d: loss %.7f %.7f, gradient %.2e" % (n_hidden, hidden, loss, l2.item(), e))
    assert abs(l2.item() - loss) <= 5e-5 * loss
    assert e <= 5e-5


@pytest.mark.parametrize("density", [False, True])
@pytest.mark.parametrize("dtype", [am.AMNERF_F32, am.AMNERF_BF16])
def test_samples_behind_a_stop_count_for_nothing(dtype, density):
    """One leaf's colours (and density) are NaN, behind opaque leaves for some rays.  A ray that stops before it
    gives the bits it gives with finite colours there: in a full launch (beside rays that march
    on), alone, and in rounds; its gradient too.  Every ray that reaches the leaf is counted."""
    scene = small_scene(s_max=192)
    at = synth.sigma_bias_offset(scene.cfg.n_hidden, scene.cfg.hidden)
    W = scene.W.copy()
    W[1:5, at] = 300.0                        # opaque: a ray stops within a few samples
    W[5:, at] = -9.0                          # all but empty
    bad = W.copy()
    bad[0, at if density else at + 1:at + 4] = np.nan
    scene.W = W
    ctx, tree, mlp = gpu_setup(scene, dtype)
    master = to_dev(bad)
    mlp_bad = am.Mlp(ctx, master, scene.cfg.n_hidden, scene.cfg.hidden, dtype, scene.n_sets)
    o, d = synth.random_rays(4000, 15)
    od, dd = to_dev(o), to_dev(d)
    ref, st, used, off = ert.render(ctx, tree, mlp, od, dd, 192, 0)
    assert st["n_nonfinite"] == 0
    _, ins = fetch_inspect(ctx, 4000, scene.n_sets)
    slot = np.repeat(ins["iv_slot"], ins["iv_n"])
    first = np.array([np.append(np.flatnonzero(slot[off[r]:off[r + 1]] == 0), 1 << 20)[0] for r in range(4000)])
    clean = used <= first
    behind = np.flatnonzero(clean & (first < 1 << 20))
    print("rays that stop before the leaf %d, that reach it %d" % (len(behind), (~clean).sum()), flush=True)
    assert len(behind) > 100 and (~clean).sum() > 100
    pick = torch.from_numpy(clean).to("cuda:0")
    for flags in (0, am.AMNERF_ERT_ROUNDS):
        out, st, used2, _ = ert.render(ctx, tree, mlp_bad, od, dd, 192, flags)
        assert np.array_equal(used2[clean], used[clean])
        assert st["n_nonfinite"] == (~clean).sum(), flags
        for k in range(3):
            assert torch.equal(out[k][pick], ref[k][pick]), (flags, k)
    for r in behind[::len(behind) // 20]:
        for flags in (0, am.AMNERF_ERT_ROUNDS):
            out = ert.render(ctx, tree, mlp_bad, od[:, r:r + 1].contiguous(), dd[:, r:r + 1].contiguous(), 192, flags)[0]
            for k in range(3):
                assert torch.equal(out[k][0], ref[k][r]), (r, flags, k)
    oc, dc = od[:, pick].contiguous(), dd[:, pick].contiguous()
    n = oc.shape[1]
    rng = np.random.default_rng(16)
    g = [to_dev(rng.standard_normal(s).astype(np.float32)) for s in ((n, 3), n, n)]
    grads = []
    for m in (mlp, mlp_bad):
        rgb = torch.empty((n, 3), device="cuda:0")
        am.amnerf_render(ctx.h, tree.h, m.desc, oc, dc, 192, rgb)
        grad = torch.empty_like(master)
        am.amnerf_render_backward(ctx.h, tree.h, m.desc, oc, dc, g[0], grad, g[1], g[2])
        grads.append(grad)
    torch.cuda.synchronize()
    assert torch.isfinite(grads[0]).all() and grads[0].abs().max() > 0
    assert torch.equal(grads[0], grads[1])


@pytest.mark.parametrize("dtype", [am.AMNERF_F32, am.AMNERF_BF16])
def test_backward_recorded_in_a_graph(dtype):
    """A backward pass recorded after an eager one, replayed after renders of other rays whose
    leaf MLPs read sorted intervals (plain) or sample records (jittered, in rounds): the gradient
    of an eager backward of the same render each time, also after a render in the static
    workspace."""
    scene = small_scene(s_max=96)
    ctx, tree, mlp = gpu_setup(scene, dtype)
    master = to_dev(scene.W)
    n = 1500
    o, d = (to_dev(a) for a in synth.random_rays(n, 19))
    g = to_dev(np.random.default_rng(20).standard_normal((n, 3)).astype(np.float32))
    rgb, eager, replayed = torch.empty((n, 3), device="cuda:0"), torch.empty_like(master), torch.empty_like(master)

    def render(**kw):
        am.amnerf_render(ctx.h, tree.h, mlp.desc, o, d, 96, rgb, **kw)

    def backward(grad):
        am.amnerf_render_backward(ctx.h, tree.h, mlp.desc, o, d, g, grad)

    render(ert_rounds=True)   # the largest workspace of these: it must not move once recorded
    render()
    backward(eager)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        backward(replayed)
    seen = []
    for k, kw in enumerate([{}, {}, dict(jitter=True, seed=5), {}, dict(ert_rounds=True), {}]):
        for t, a in zip((o, d), synth.random_rays(n, 30 + k)):
            t.copy_(to_dev(a))
        print("replay after a render with", kw, flush=True)
        render(**kw)
        replayed.fill_(-1.0)
        graph.replay()
        torch.cuda.synchronize()
        backward(eager)
        torch.cuda.synchronize()
        assert torch.isfinite(eager).all() and torch.equal(replayed, eager), (k, kw)
        seen.append(eager.clone())
        am.amnerf_render_static(ctx.h, tree.h, mlp.desc, o[:, :300].contiguous(), d[:, :300].contiguous(), 96, rgb)
        replayed.fill_(-1.0)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(replayed, eager), (k, kw, "after a render elsewhere")
    assert not torch.equal(seen[0], seen[1])


def pair_crossing(s, o, d):
    """(s - o) / d as a float32 pair by division: TwoSum of the numerator, the division's exact
    remainder (float64 holds it: two 24-bit factors), its quotient, normalised."""
    s, o, d = (np.asarray(a, np.float32) for a in (s, o, d))
    hi = s - o
    bb = hi - s
    lo = (s - (hi - bb)) + (-o - bb)
    q0 = hi / d
    r = (hi.astype(np.float64) - q0.astype(np.float64) * d.astype(np.float64)).astype(np.float32) + lo
    q1 = r / d
    h = q0 + q1
    return h, q1 - (h - q0)


def pair_pick(pairs, largest):
    """Per element the largest or smallest of float pairs (high parts, then low parts)."""
    h, l = pairs[0]
    for a, b in pairs[1:]:
        take = (h < a) | ((h == a) & (l < b)) if largest else (a < h) | ((a == h) & (b < l))
        h, l = np.where(take, a, h), np.where(take, b, l)
    return h, l


def test_crossings_have_the_bits_of_a_division():
    """The first interval of each ray, from inside the box to 2^18 away: entry and length bit for
    bit those of crossings formed by division (later intervals take their exit from the stack,
    whose low parts are shorter)."""
    scene = small_scene(max_leaves=64, max_depth=9, s_max=33)
    ctx, tree, mlp = gpu_setup(scene, am.AMNERF_F32)
    rng = np.random.default_rng(14)
    n = 60000
    u = rng.standard_normal((3, n))
    u /= np.linalg.norm(u, axis=0)
    dist = 2.0 ** rng.uniform(-2, 18, n)
    tgt = rng.uniform(0.05, 0.95, (3, n))
    o = (tgt + u * dist).astype(np.float32)
    d = (tgt - o.astype(np.float64))
    d = (d / np.linalg.norm(d, axis=0)).astype(np.float32)
    assert (np.abs(d) > 2.0 ** -100).all()
    render_all(scene, ctx, tree, mlp, o, d, 33)
    _, ins = fetch_inspect(ctx, n, scene.n_sets)
    off = ins["ray_iv_off"].astype(np.int64)
    r = np.flatnonzero(np.diff(off) > 0)
    i = off[r]
    o, d = o[:, r], d[:, r]
    boxes = scene.otree.leaf_boxes()[ins["iv_slot"][i]].astype(np.float32) / np.float32(scene.cfg.grid_n)
    near, far = [(np.zeros(len(r), np.float32),) * 2], []
    for a in range(3):
        near.append(pair_crossing(np.where(d[a] > 0, 0.0, 1.0), o[a], d[a]))
        far.append(pair_crossing(np.where(d[a] > 0, boxes[:, 3 + a], boxes[:, a]), o[a], d[a]))
    t0, l0 = pair_pick(near, True)
    t1, l1 = pair_pick(far, False)
    dt = (t1 - t0) + (l1 - l0)
    print("rays %d, of them more than 2^12 away %d; other lengths %d" % (
        len(r), (t0 > 4096).sum(), (ins["iv_dt"][i] != dt).sum()), flush=True)
    assert (t0 > 4096).sum() > 500 and (t0 == 0).sum() > 500
    assert np.array_equal(ins["iv_t0"][i], t0)
    assert np.array_equal(ins["iv_dt"][i], dt)


@pytest.mark.parametrize("tiny", [1.4e-45, 1e-39, 5e-39, 1.17e-38, 2e-38])
def test_tiny_direction_components(tiny):
    """Components down to the smallest there is: the intervals are those of a component of zero
    (the ray moves less than 1e-37 along it), the other planes' crossings the same to the bit."""
    scene = small_scene(s_max=33)
    ctx, tree, mlp = gpu_setup(scene, am.AMNERF_F32)
    o, d = synth.random_rays(600, 4)
    for r in range(0, 600, 3):
        d[r % 9 // 3, r] = 0.0
    small = d.copy()
    for r in range(0, 600, 3):
        small[r % 9 // 3, r] = np.float32(tiny) * (1 if r % 2 else -1)
    got = []
    for dd in (d, small):
        render_all(scene, ctx, tree, mlp, o, dd, 33)
        got.append(fetch_inspect(ctx, 600, scene.n_sets)[1])
    for k in ("ray_iv_off", "iv_slot", "iv_n", "iv_t0", "iv_dt"):
        assert np.array_equal(got[0][k], got[1][k]), k


@pytest.mark.parametrize("backward", [False, True])
def test_a_workspace_cap_decides_the_row_source_not_the_result(backward):
    """Under a workspace cap a render takes the layout with sorted intervals only where it fits a
    workspace made for sample records: with 255 samples per ray, the cap that a jittered render
    (which has records in any case), or one and its backward, just fit is enough without jitter
    too, and the bits are those of a context without a cap."""
    scene = Scene(synth.scaled(synth.C2, grid_n=64, max_leaves=300, max_depth=12, n_hidden=2, hidden=32))
    assert scene.n_sets >= 255
    o, d = (to_dev(a) for a in synth.random_rays(3000, 17))
    W = to_dev(scene.W)
    g = torch.ones((3000, 3), device="cuda:0")

    def run(cap, jitter):
        ctx = am.Context(0, cap)
        tree = am.Tree(ctx, scene.grid, scene.cfg.grid_n, scene.cfg.max_depth, scene.cfg.max_leaves)
        mlp = am.Mlp(ctx, W, 2, 32, am.AMNERF_BF16, scene.n_sets)
        rgb, grad = torch.empty((3000, 3), device="cuda:0"), torch.zeros_like(W)
        try:
            am.amnerf_render(ctx.h, tree.h, mlp.desc, o, d, 255, rgb, jitter=jitter)
            if backward:
                am.amnerf_render_backward(ctx.h, tree.h, mlp.desc, o, d, g, grad)
        except am.AmnerfError as e:
            assert e.code == am.AMNERF_ENOMEM
            return None
        torch.cuda.synchronize()
        return rgb, grad

    lo, hi = 1 << 20, 1 << 31
    while hi - lo > 1 << 12:
        mid = (lo + hi) // 2
        if run(mid, True) is None:
            lo = mid
        else:
            hi = mid
    print("records fit %d bytes" % hi, flush=True)
    free = run(0, False)
    for cap in (hi, hi + (hi >> 6), hi + (hi >> 4), 2 * hi):
        got = run(cap, False)
        assert got is not None, cap
        assert torch.equal(got[0], free[0]) and torch.equal(got[1], free[1]), cap


def test_static_render_where_only_records_fit():
    """Rays between the largest static call on sorted intervals and the largest on sample
    records: the bits of the same render in the context's own workspace."""
    scene = Scene(synth.scaled(synth.C2, grid_n=64, max_leaves=300, max_depth=12, n_hidden=2, hidden=32))
    ctx, tree, mlp = gpu_setup(scene, am.AMNERF_BF16)
    # per ray 36 bytes per interval and 28 per sample; 40 per interval with the intervals' records
    n = int(am.amnerf_render_static_capacity() / (40 * 255 + 28 * 255)) + 40
    o, d = (to_dev(a) for a in synth.random_rays(n, 18))
    a, _, _, _ = ert.render(ctx, tree, mlp, o, d, 255, 0, static=True)
    b, _, _, _ = ert.render(ctx, tree, mlp, o, d, 255, 0)
    ert.compare(a, b, n)
