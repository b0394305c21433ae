"""The view-dependent MLP's backward by groups of 16 rays, eight groups a
workgroup, a bounded number of workgroups: batches around a group, around a
workgroup, and of several groups a wave, against the oracle's float64
adjoint."""
import numpy as np
import pytest

import synth
from oracle import sh

from helpers import gpu_renderer, scene_and_dist, to_gpu

pytestmark = pytest.mark.gpu


def _inputs(sc):
    """Rays none of whose hidden units lies within 1e-4 of its kink, where
    float32 and float64 may take different sides."""
    rng = np.random.default_rng(21)
    c_d = rng.normal(size=(700, 3)).astype(np.float32)
    feat = rng.normal(size=(700, 4)).astype(np.float32)
    d = rng.normal(size=(700, 3)).astype(np.float32)
    d[5] = 0.0                                       # no direction: SH = 0
    p = sc.mlp.astype(np.float64)
    W0, b0 = p[:64 * 23].reshape(64, 23), p[64 * 23:64 * 24]
    W1, b1 = p[64 * 24:64 * 88].reshape(64, 64), p[64 * 88:64 * 89]
    x = np.concatenate([c_d, feat, sh.sh16(d)], axis=1).astype(np.float64)
    z1 = x @ W0.T + b0
    z2 = np.maximum(z1, 0.0) @ W1.T + b1
    keep = (np.abs(z1).min(1) > 1e-4) & (np.abs(z2).min(1) > 1e-4)
    assert keep.sum() >= 300
    return c_d[keep], feat[keep], d[keep]


@pytest.mark.parametrize("n", [1, 15, 16, 17, 127, 128, 129, 4099, 33001, 70000])
def test_batches_around_groups_and_workgroups(n):
    import torch
    print(f"[view mlp backward] {n} rays", flush=True)
    sc, _ = scene_and_dist("tiny_view")
    base = _inputs(sc)
    idx = np.arange(n) % len(base[0])
    c_d, feat, d = (a[idx] for a in base)
    g = np.random.default_rng(n).normal(size=(n, 3)).astype(np.float32)
    r = gpu_renderer("tiny_view")
    gd, gc, gf, gg = to_gpu(d, c_d, feat, g)
    gm = torch.full((r.n_mlp,), 0.5, device="cuda")              # added to, not overwritten
    gcf = r.view_mlp_backward(gd, gc, gf, gg, gm).cpu().numpy()
    w_cd, w_f, w_p = sh.mlp_view_backward64(sc.mlp, c_d.astype(np.float64), feat.astype(np.float64), d,
                                            g.astype(np.float64))
    want = np.concatenate([w_cd, w_f], axis=1)
    # chains of at most 64 float32 products and sums, a relative 1e-5 of the
    # largest with room; the weight gradients also sum n rays
    assert np.abs(gcf - want).max() <= 1e-4 * np.abs(want).max()
    assert np.abs((gm.cpu().numpy() - 0.5) - w_p).max() <= 1e-4 * max(np.abs(w_p).max(), 0.5)
    again = torch.full((r.n_mlp,), 0.5, device="cuda")
    r.view_mlp_backward(gd, gc, gf, gg, again)
    assert torch.equal(gm, again)                                # a fixed order of sums
