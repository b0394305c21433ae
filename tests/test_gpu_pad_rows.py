"""The backward's padded gradient rows: an optional buffer beside its
workspace.

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


def _lib():
    from paper_2407_10482_amd._lib import load_library
    return load_library()


@pytest.fixture(autouse=True)
def _disarm():
    yield
    _lib().ngprt_test_fail_alloc(-1)


def _rays(name, n):
    cfg = scene_and_dist(name)[0].cfg
    cams = synth.random_sphere_cameras(5, 1.0, seed=61)
    o, d, _ = synth.scene_rays(cfg, cams=cams, width=64, height=64)
    g = np.random.default_rng(1).standard_normal((len(o), 3)).astype(np.float32)
    return to_gpu(o[:n], d[:n], g[:n])


def _grads(r, o, d, g):
    """The batch's gradients: tables, MLP and, for the baked model, the atlas."""
    import torch
    gt, gm = torch.zeros((r.L, r.T, 9), device="cuda"), torch.zeros((r.n_mlp,), device="cuda")
    if r.feature_model:
        ga = torch.zeros((r.n_blocks, 8, 8, 8, 8 + 2 * r.L), device="cuda")
        r.backward_baked(o, d, g, gt, ga, gm)
        return gt, gm, ga
    r.backward(o, d, g, gt, gm)
    return gt, gm


def _close(a, b):
    return float((a.double() - b.double()).norm()) <= TOL * float(b.double().norm())


# batches that pad the tables' rows (2^14 a level: from 1,024 rays on)
@pytest.mark.parametrize("name,n", [("tiny", 1024), ("tiny", 16500), ("baked_tiny", 16500)])
def test_no_memory_for_padded_rows(name, n):
    """With the workspace at hand and no memory for the padded rows the call
    scatters into the caller's rows; a later call may pad again."""
    from paper_2407_10482_amd._lib import NgprtError
    print(f"[no padded rows {name} {n}]", flush=True)
    o, d, g = _rays(name, n)
    want = _grads(gpu_renderer(name), o, d, g)
    r = gpu_renderer(name)
    # the deterministic mode takes the workspace and no padded rows (the baked
    # model refuses it, with the workspace taken)
    r.set_deterministic(True)
    if r.feature_model:
        with pytest.raises(NgprtError, match="UNSUPPORTED"):
            _grads(r, o, d, g)
    else:
        _grads(r, o, d, g)
    r.set_deterministic(False)
    for _ in range(2):
        _lib().ngprt_test_fail_alloc(0)
        got = _grads(r, o, d, g)
        assert all(float(b.abs().max()) > 0 and _close(a, b) for a, b in zip(got, want))
    _lib().ngprt_test_fail_alloc(-1)
    got = _grads(r, o, d, g)
    assert all(_close(a, b) for a, b in zip(got, want))
