"""The float32 leaf MLPs sample by sample against float64, over the shapes of both kernels
(split values on the bfloat16 matrix cores up to 7 layers of 64, float32 instructions above)
and bucket sizes from one sample to several tiles with remainders."""
import numpy as np
import pytest
import torch

import synth
from scene_util import Scene, gpu_setup, to_dev

pytestmark = pytest.mark.gpu


def _features(p, d):
    f = [p]
    for k in range(4):
        f += [np.sin(np.pi * 2.0 ** k * p), np.cos(np.pi * 2.0 ** k * p)]
    return np.concatenate(f + [d], axis=1)


@pytest.mark.parametrize("n_hidden,hidden,n_rays", [(1, 32, 1), (2, 32, 37), (8, 32, 300), (1, 64, 3), (4, 64, 500),
                                                    (7, 64, 65), (8, 64, 65)])
def test_float32_outputs_per_sample(n_hidden, hidden, n_rays):
    """Bar: inputs within 2 ulp of the features, and per layer at most 8 roundings of sums whose
    terms are of the output's size, so a sample's error is below about (2 + 8 (n_hidden + 1))
    2^-24 of the layer's largest values (4 rms): 16 (n_hidden + 2) 2^-24 of the rms, times 2."""
    import paper_2310_01881_amd as am
    cfg = synth.scaled(synth.C1, n_hidden=n_hidden, hidden=hidden, max_leaves=7, s_max=33)
    scene = Scene(cfg)
    rng = np.random.Generator(np.random.PCG64(5))
    scene.W = (scene.W + 0.05 * rng.standard_normal(scene.W.shape)).astype(np.float32)   # biases too
    ctx, tree, mlp = gpu_setup(scene, am.AMNERF_F32)
    o, d = synth.random_rays(n_rays, 11)
    od, dd = to_dev(o), to_dev(d)
    am.render(ctx, tree, mlp, od, dd, cfg.s_max)
    st = am.amnerf_render_stats_get(ctx.h)
    ni, ns = st["n_intervals"], st["n_samples"]
    assert ns > 0
    buf = {k: torch.empty(n, dtype=t, device="cuda") for k, n, t in
           [("ray_iv_off", n_rays + 1, torch.int32), ("iv_t0", ni, torch.float32), ("iv_dt", ni, torch.float32),
            ("iv_slot", ni, torch.int32), ("iv_n", ni, torch.int32), ("sample_out", 4 * ns, torch.float32)]}
    am.amnerf_render_inspect(ctx.h, **buf)
    h = {k: v.cpu().numpy() for k, v in buf.items()}
    n = h["iv_n"]
    which = np.repeat(np.arange(ni), n)
    j = np.arange(ns) - np.repeat(np.cumsum(n) - n, n)
    ray = np.repeat(np.arange(n_rays), np.diff(h["ray_iv_off"]))[which]
    # the kernels' own float32 positions (one rounding per fused step), then float64
    delta = (h["iv_dt"] / n.astype(np.float32))[which].astype(np.float64)
    t = ((j + 0.5) * delta + h["iv_t0"][which].astype(np.float64)).astype(np.float32).astype(np.float64)
    dr, orr = d.T[ray].astype(np.float64), o.T[ray].astype(np.float64)
    x = (t[:, None] * dr + orr).astype(np.float32).astype(np.float64)
    p = (2.0 * x - 1.0).astype(np.float32).astype(np.float64)
    f = _features(p, dr)
    slot = h["iv_slot"][which]
    z = np.empty((ns, 4))
    for s in np.unique(slot):
        a, off = f[slot == s], 0
        for l, (fi, fo) in enumerate(synth.layer_dims(n_hidden, hidden)):
            w = scene.W[s].astype(np.float64)
            a = a @ w[off:off + fi * fo].reshape(fo, fi).T + w[off + fi * fo:off + fi * fo + fo]
            off += fi * fo + fo
            if l < n_hidden:
                a = np.maximum(a, 0.0)
        z[slot == s] = a
    err = np.abs(h["sample_out"].reshape(-1, 4) - z).max() / np.sqrt((z * z).mean())
    print("%d x %d: max error / rms %.2e" % (n_hidden, hidden, err))
    assert err < 32 * (n_hidden + 2) * 2.0 ** -24


def _sample_outputs(ctx, n_rays):
    """(leaf, ray, pre-activations) of the last render's samples, and its statistics."""
    import paper_2310_01881_amd as am
    st = am.amnerf_render_stats_get(ctx.h)
    ni, ns = st["n_intervals"], st["n_samples"]
    assert ns > 0
    buf = {k: torch.empty(n, dtype=t, device="cuda") for k, n, t in
           [("ray_iv_off", n_rays + 1, torch.int32), ("iv_slot", ni, torch.int32), ("iv_n", ni, torch.int32),
            ("sample_out", 4 * ns, torch.float32)]}
    am.amnerf_render_inspect(ctx.h, **buf)
    h = {k: v.cpu().numpy() for k, v in buf.items()}
    ray = np.repeat(np.arange(n_rays), np.diff(h["ray_iv_off"]))
    return np.repeat(h["iv_slot"], h["iv_n"]), np.repeat(ray, h["iv_n"]), h["sample_out"].reshape(-1, 4), st


def _blocks(W, n_hidden, hidden):
    """Views of a parameter array: per layer the weights [set][out][in] and the biases."""
    out, off = [], 0
    for fi, fo in synth.layer_dims(n_hidden, hidden):
        out.append((W[:, off:off + fi * fo].reshape(len(W), fo, fi), W[:, off + fi * fo:off + fi * fo + fo]))
        off += fi * fo + fo
    return out


DIR = 27   # the first input that is the ray's direction, as it was given


@pytest.mark.parametrize("n_hidden,hidden", [(1, 32), (2, 64), (4, 64), (8, 64)])
@pytest.mark.parametrize("case", ["overflow", "infinite", "nan", "largest"])
def test_values_that_are_not_finite(case, n_hidden, hidden):
    """Hidden sums that overflow, infinite, NaN and largest finite weights: every pre-activation
    is the infinity or NaN that float32 arithmetic gives (a ReLU of NaN is 0), finite ones to
    1e-6 of their size, and the rays are counted.  The last shape runs on the float32
    instructions."""
    import paper_2310_01881_amd as am
    cfg = synth.scaled(synth.C1, n_hidden=n_hidden, hidden=hidden, max_leaves=8, s_max=17)
    scene = Scene(cfg)
    rng = np.random.default_rng(22)
    n_rays, L = 200, scene.n_sets
    d = (np.array([[0.7], [0.6], [0.4]]) + rng.uniform(-0.05, 0.05, (3, n_rays))).astype(np.float32)
    o = (0.5 - 1.5 * d + rng.uniform(-0.2, 0.2, d.shape)).astype(np.float32)
    scene.W = np.zeros_like(scene.W)
    b = _blocks(scene.W, n_hidden, hidden)
    w0, b0 = b[0]
    w0[:, :, DIR:DIR + 3] = rng.uniform(0.1, 1.0, (L, hidden, 3))     # every unit positive
    for l in range(1, n_hidden):
        b[l][0][:] = rng.uniform(0.1, 1.0, (L, hidden, hidden)) / hidden
    wo = b[n_hidden][0]
    wo[:] = rng.uniform(-1.0, 1.0, wo.shape)
    wo[:, 0] = np.abs(wo[:, 0])                                       # density: positive
    k = 5                                                             # the unit in question
    if case == "overflow":
        w0[:, k, DIR:DIR + 2] = 3e38
    elif case == "infinite":
        w0[:, k, DIR] = np.inf
        w0[:, k + 1, DIR + 1] = -np.inf                               # off
        if n_hidden > 1:
            b[1][0][:, 3, k + 1] = np.inf                             # an infinite weight of an input of 0
    elif case == "nan":
        w0[:, k, DIR] = np.nan                                        # off
        if n_hidden > 1:
            b[1][0][:, 2, 7] = np.nan
        wo[:, 0, 1] = np.inf
    else:
        w0[:, k, DIR:DIR + 3] = (np.float32(3.4028234e38) * np.float32(0.9999), 0.0, 0.0)
        for l in range(1, n_hidden + 1):
            b[l][0][:, :, k] = 0.0
        if n_hidden > 1:
            b[1][0][:, 0, k] = 1e-30
        else:
            wo[:, 1, k] = 1e-30
    ctx, tree, mlp = gpu_setup(scene, am.AMNERF_F32)
    am.render(ctx, tree, mlp, to_dev(o), to_dev(d), cfg.s_max)
    slot, ray, z, st = _sample_outputs(ctx, n_rays)
    ref = np.empty((L, n_rays, 4), np.float32)
    with np.errstate(all="ignore"):
        for s in range(L):
            a = np.zeros((n_rays, 30), np.float64)                    # (weights of positions are 0)
            a[:, DIR:DIR + 3] = d.T
            for l in range(n_hidden + 1):
                wl, bl = b[l][0][s].astype(np.float64), b[l][1][s].astype(np.float64)
                a = ((a[:, None, :] * wl[None]).sum(axis=2) + bl).astype(np.float32)
                if l < n_hidden:
                    a = np.fmax(a, 0.0).astype(np.float64)
            ref[s] = a
    want = ref[slot, ray]
    odd = ~np.isfinite(want)
    print("%s %dx%d: %d of %d values not finite, %d rays counted" % (
        case, n_hidden, hidden, odd.sum(), odd.size, st["n_nonfinite"]), flush=True)
    assert odd.any() == (case != "largest")
    assert np.array_equal(np.isnan(z), np.isnan(want))
    assert np.array_equal(np.isposinf(z), np.isposinf(want)) and np.array_equal(np.isneginf(z), np.isneginf(want))
    np.testing.assert_allclose(z[~odd], want[~odd], rtol=0, atol=1e-6 * max(1.0, np.abs(want[~odd]).max(initial=0.0)))
    assert (st["n_nonfinite"] > 0) == odd.any()


@pytest.mark.parametrize("n_hidden,hidden,layer", [(1, 32, 0), (1, 64, 0), (3, 32, 1), (4, 64, 2), (7, 64, 6), (8, 64, 3)])
def test_a_product_keeps_its_24_bits(n_hidden, hidden, layer):
    """Each output is one product w x (x a component of the direction, the other layers passing it
    on unchanged), for values whose low bits are all set and random ones.  Bar: one rounding of
    the result, and eight of sums below 2^-6 of it: 2^-24 (1 + 2^-3)."""
    import paper_2310_01881_amd as am
    cfg = synth.scaled(synth.C1, n_hidden=n_hidden, hidden=hidden, max_leaves=8, s_max=17)
    scene = Scene(cfg)
    rng = np.random.default_rng(21)
    n_rays, L = 400, scene.n_sets
    x = rng.uniform(0.25, 1.0, (3, n_rays)).astype(np.float32)
    x[:, ::2] = np.float32(0.5) * np.float32(1 + 2.0 ** -7 - 2.0 ** -23)
    x[1, ::4] = np.float32(1 - 2.0 ** -24)
    x[2, ::8] = np.float32(0.5) * np.float32(1 + 2.0 ** -8 - 2.0 ** -23)
    w = rng.uniform(0.5, 2.0, (L, hidden)).astype(np.float32)
    w[:, ::2] = np.float32(1 + 2.0 ** -8 - 2.0 ** -16 + 2.0 ** -17 - 2.0 ** -23)
    w[1::2, 1] = np.float32(2 - 2.0 ** -23)
    w[:, 2] = np.float32(1 + 2.0 ** -8 + 2.0 ** -17 - 2.0 ** -23)
    scene.W = np.zeros_like(scene.W)
    b = _blocks(scene.W, n_hidden, hidden)
    for l in range(n_hidden):
        for j in range(hidden):
            b[l][0][:, j, DIR + j % 3 if l == 0 else j] = w[:, j] if l == layer else 1.0
    units = rng.integers(0, hidden, (L, 4))
    units[:, :3] = (0, 1, 2)
    for s in range(L):
        for k in range(4):
            b[n_hidden][0][s, k, units[s, k]] = 1.0
    ctx, tree, mlp = gpu_setup(scene, am.AMNERF_F32)
    o = (0.5 - 1.5 * x + rng.uniform(-0.2, 0.2, x.shape)).astype(np.float32)
    am.render(ctx, tree, mlp, to_dev(o), to_dev(x), cfg.s_max)
    slot, ray, z, _ = _sample_outputs(ctx, n_rays)
    u = units[slot]
    ref = w[slot[:, None], u].astype(np.float64) * x[u % 3, ray[:, None]].astype(np.float64)
    e = np.abs(z - ref) / ref
    print("%d x %d, layer %d: %d products, largest relative error 2^%.2f, rms 2^%.2f" % (
        n_hidden, hidden, layer, e.size, np.log2(e.max()), np.log2(np.sqrt((e * e).mean()))))
    assert e.max() <= 2.0 ** -24 * (1 + 2.0 ** -3)
