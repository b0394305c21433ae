"""Backward batches above 16,384 rays (four lanes a ray) against the same rays
in parts of fewer (sixteen lanes a ray, which the oracle tests check): the
distortion regulariser's prefix sums, the contracted march with and without a
pyramid, and the MLP gradient's partial sums.

Tolerance: the two sides add the same float32 contributions in another order; a
sum of m terms is off by about eps sqrt(m) of its terms' size, and no entry
here gets more than 5e4: 6e-8 * sqrt(5e4) = 1.3e-5, taken as 2e-5 in the norm.
"""
import numpy as np
import pytest

import synth
from helpers import gpu_renderer, scene_and_dist, to_gpu

pytestmark = pytest.mark.gpu
TOL = 2e-5
CONTRACT = dict(domain=synth.configs.DOMAIN_CONTRACT, roi_half=2.0, step=float(synth.CONTRACT_STEP))


def _rays(name, contract, n):
    cfg = scene_and_dist(name)[0].cfg
    if name == "hd":
        o, d, _ = synth.scene_rays(cfg, cams=synth.camera_positions(cfg)[:3], width=96, height=64)
    else:
        cams = synth.random_sphere_cameras(5, 2.5 if contract else 1.0, seed=51)
        o, d, _ = synth.scene_rays(cfg, cams=cams, width=64, height=64)
    g = np.random.default_rng(2).standard_normal((len(o), 3)).astype(np.float32)
    assert n <= len(o)
    return to_gpu(o[:n], d[:n], g[:n])


@pytest.mark.parametrize("n", [16385, 16500])
@pytest.mark.parametrize("name,contract,dist", [("tiny", False, False), ("tiny", False, True), ("hd", False, False),
                                                ("hd", False, True), ("tiny_pyramid", True, True),
                                                ("baked_tiny", True, False), ("baked_tiny_pyramid", True, True),
                                                ("baked_tiny_l3", False, True)])
def test_whole_batch_against_parts(name, contract, dist, n):
    import torch
    print(f"[batch {name} contracted {contract} dist {dist} n {n}]", flush=True)
    r = gpu_renderer(name, **(CONTRACT if contract else {}))
    o, d, g = _rays(name, contract, n)
    # per ray, so that a sum over the wrong ray's samples shows
    gdist = torch.linspace(0.01, 0.05, n, device="cuda") if dist else None
    baked = bool(r.feature_model)

    def grads(edges):
        shapes = [(r.L, r.T, 9), (r.n_mlp,)] + ([(r.n_blocks, 8, 8, 8, 8 + 2 * r.L)] if baked else [])
        out = [torch.zeros(s, device="cuda") for s in shapes]
        for lo, hi in zip(edges, edges[1:]):
            a = [x[lo:hi].contiguous() for x in (o, d, g)]
            gd = gdist[lo:hi].contiguous() if dist else None
            if baked:
                r.backward_baked(*a, out[0], out[2], out[1], gd)
            else:
                r.backward(*a, out[0], out[1], gd)
        return out
    assert int(r.render(o, d)["n_samples"].max()) > 16
    for a, b in zip(grads([0, n]), grads([0, 7, 300, 9001, n])):
        assert float(b.abs().max()) > 0
        assert float((a.double() - b.double()).norm()) <= TOL * float(b.double().norm())


@pytest.mark.parametrize("name", ["paper_tiny", "tiny_view"])
def test_given_feature_gradients_with_regulariser(name):
    """The same through ngprt_render_backward_features (the view-dependent
    MLP's path), contracted."""
    import torch
    print(f"[batch {name}, feature gradients + dist]", flush=True)
    n = 16500
    r = gpu_renderer(name, **CONTRACT)
    o, d, _ = _rays(name, True, n)
    cf = torch.from_numpy(np.random.default_rng(4).standard_normal((n, 7)).astype(np.float32)).cuda()
    gdist = torch.linspace(0.01, 0.05, n, device="cuda")
    baked = bool(r.feature_model)

    def grads(edges):
        out = [torch.zeros((r.L, r.T, 9), device="cuda")]
        if baked:
            out.append(torch.zeros((r.n_blocks, 8, 8, 8, 8 + 2 * r.L), device="cuda"))
        for lo, hi in zip(edges, edges[1:]):
            o1, d1, c1, g1 = (x[lo:hi].contiguous() for x in (o, d, cf, gdist))
            r.backward_features(o1, d1, c1, out[0], out[1] if baked else None, g1)
        return out
    for a, b in zip(grads([0, n]), grads([0, 63, 8000, n])):
        assert float(b.abs().max()) > 0
        assert float((a.double() - b.double()).norm()) <= TOL * float(b.double().norm())
