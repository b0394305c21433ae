"""The backward's merged scatter where its paths change: batch sizes around the
lanes-a-ray and padded-row rules and ragged workgroups, waves whose samples
share every cell, non-finite gradients.  The reference is the library's
deterministic mode (one record per contribution, no merging) or, for the baked
model, the same batch taken in parts.

Tolerance: both sides add the same float32 contributions in another order; a
sum of m terms is off by about eps sqrt(m) of its terms' size, and no entry
here gets more than 5e4: 6e-8 * sqrt(5e4) = 1.3e-5, taken as 2e-5 in the norm.
"""
import numpy as np
import pytest

import synth
from helpers import gpu_renderer, scene_and_dist, to_gpu

pytestmark = pytest.mark.gpu
TOL = 2e-5


def _rays(name, n, seed=0):
    cfg = scene_and_dist(name)[0].cfg
    cams = synth.random_sphere_cameras(5, 1.0, seed=40 + seed)
    o, d, _ = synth.scene_rays(cfg, cams=cams, width=64, height=64)
    g = np.random.default_rng(seed).standard_normal((len(o), 3)).astype(np.float32)
    assert n <= len(o)
    return to_gpu(o[:n], d[:n], g[:n])


def _hash_grads(r, o, d, g, gdist=None):
    import torch
    gt = torch.zeros((r.L, r.T, 9), device="cuda")
    gm = torch.zeros((r.n_mlp,), device="cuda")
    r.backward(o, d, g, gt, gm, gdist)
    return gt, gm


def _close(a, b):
    return float((a.double() - b.double()).norm()) <= TOL * float(b.double().norm())


@pytest.mark.parametrize("n", [1, 15, 17, 255, 1023, 1024, 4097, 16384, 16385])
def test_against_deterministic_mode(n):
    import torch
    print(f"[scatter n {n}]", flush=True)
    r = gpu_renderer("tiny")
    o, d, g = _rays("tiny", n)
    gdist = torch.full((n,), 1e-3, device="cuda") if n in (17, 4097) else None
    gt, gm = _hash_grads(r, o, d, g, gdist)
    if n > 4097:                              # the records of a whole batch exceed their limit: in parts
        want = torch.zeros_like(gt)
        r.set_deterministic(True)
        for lo in range(0, n, 4096):
            s = slice(lo, min(lo + 4096, n))
            want += _hash_grads(r, o[s].contiguous(), d[s].contiguous(), g[s].contiguous())[0]
    else:
        r.set_deterministic(True)
        want, gm2 = _hash_grads(r, o, d, g, gdist)
        assert torch.equal(gm, gm2)           # the MLP gradient bit for bit in both modes
    assert _close(gt, want)
    assert bool(((gt != 0).any(2) == (want != 0).any(2)).float().mean() > 0.9999)


def test_one_ray_repeated():
    """Every wave's samples share every cell of every level."""
    import torch
    print("[scatter repeated ray]", flush=True)
    r = gpu_renderer("tiny")
    o, d, g = _rays("tiny", 4096)
    out = r.render(o, d)
    i = int(out["n_samples"].argmax())
    n = 320
    oo, dd, gg = (x[i:i + 1].expand(n, 3).contiguous() for x in (o, d, g))
    gt, _ = _hash_grads(r, oo, dd, gg)
    one, _ = _hash_grads(r, oo[:1].contiguous(), dd[:1].contiguous(), gg[:1].contiguous())
    assert _close(gt, one * n)


@pytest.mark.parametrize("n", [700, 16500])
def test_non_finite_gradients_stay_in_their_entries(n):
    import torch
    print(f"[scatter non-finite n {n}]", flush=True)
    r = gpu_renderer("tiny")
    o, d, g = _rays("tiny", n)
    ns = r.render(o, d)["n_samples"]
    hit = int((ns > 4).nonzero()[n // 40])
    g[hit, 1] = float("nan")
    gt, _ = _hash_grads(r, o, d, g)
    s = slice(hit, hit + 1)
    r.set_deterministic(True)
    alone, _ = _hash_grads(r, o[s].contiguous(), d[s].contiguous(), g[s].contiguous())
    assert bool(torch.isnan(alone).any()) and torch.equal(torch.isnan(gt), torch.isnan(alone))


@pytest.mark.parametrize("name", ["baked_tiny", "baked_tiny_l3", "baked_tiny_pyramid"])
def test_baked_whole_batch_against_parts(name):
    import torch
    print(f"[scatter {name}]", flush=True)
    r = gpu_renderer(name)
    n = 16500
    o, d, g = _rays(name, n)

    def grads(parts):
        out = [torch.zeros(s, device="cuda") for s in ((r.L, r.T, 9), (r.n_blocks, 8, 8, 8, 8 + 2 * r.L), (451,))]
        for lo, hi in parts:
            r.backward_baked(o[lo:hi].contiguous(), d[lo:hi].contiguous(), g[lo:hi].contiguous(), *out)
        return out
    whole = grads([(0, n)])
    parts = grads([(0, 7), (7, 300), (300, 9001), (9001, n)])
    for a, b in zip(whole, parts):
        assert float(b.abs().max()) > 0 and _close(a, b)
    assert float(whole[0][:, :, 8].abs().max()) == 0.0        # no logit gradient in the baked model
