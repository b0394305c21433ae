"""Renders on either side of the lanes-a-ray rule's lines (16, 8 or one lane a
ray by launch size and domain, one beyond 16,384 rays of at most three samples):
the same bits whatever the launch a ray is part of."""
import dataclasses

import numpy as np
import pytest

import synth
from helpers import gpu_renderer, scene_and_dist, to_gpu

pytestmark = pytest.mark.gpu


def _renderer(domain, dtype, max_samples):
    """The tiny scene, or its tables and occupancy in the contracted domain."""
    if domain == "box":
        return gpu_renderer("tiny", dtype, max_samples=max_samples)
    return gpu_renderer("tiny", dtype, max_samples=max_samples, domain=synth.configs.DOMAIN_CONTRACT, roi_half=2.0,
                        step=float(synth.CONTRACT_STEP))


@pytest.mark.parametrize("max_samples", [3, 4, 1024])
@pytest.mark.parametrize("domain,dtype", [("box", 0), ("box", 1), ("contract", 0), ("contract", 2)])
def test_same_bits_across_the_lines(domain, dtype, max_samples):
    import torch
    print(f"[render lanes {domain} {dtype} cap {max_samples}]", flush=True)
    cfg = scene_and_dist("tiny", dtype)[0].cfg
    cams = synth.random_sphere_cameras(21, 1.0 if domain == "box" else 2.5, seed=78)
    o, d, _ = synth.scene_rays(dataclasses.replace(cfg, cam_radius=1.0), cams=cams, width=64, height=64)
    o, d = to_gpu(o[:81921], d[:81921])
    d[7] = float("nan")
    r = _renderer(domain, dtype, max_samples)
    line = 28672 if domain == "box" else 61440

    def render(n, labels):
        out = r.alloc_outputs(n, labels=labels)
        if labels:
            out["dist_loss"] = torch.empty((n,), device="cuda")
        return r.render(o[:n].contiguous(), d[:n].contiguous(), out=out)
    for labels in (False, True):
        want = render(81921, labels)
        assert int(want["n_samples"].max()) >= min(max_samples, 17)
        for n in (17, 16384, 16385, line - 1, line, line + 1, line + 7, 81913, 81920):
            got = render(n, labels)
            for k, v in got.items():
                assert torch.equal(v.view(torch.int32), want[k][:n].contiguous().view(torch.int32)), (n, labels, k)
