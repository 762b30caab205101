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
