"""Proposal renders that march on past their far end (far_guard > 0) in the
contracted domain, against the oracle: the resumed ray visits the lattice
point that stopped it, so counts, reads and transmittance bits are the
oracle's, and so are the lattice indices of its samples (the distortion
output is a function of them)."""
import numpy as np
import pytest

from oracle import pyramid
from oracle.distgrid import distance_grid_edt
from oracle.grad import ray_distortion
from oracle.render import CONTRACT, OracleInputs, render, render_proposal
import synth

from helpers import scene_and_dist, to_gpu

pytestmark = pytest.mark.gpu
F32 = np.float32
GUARD = 1e-3


def _scene(pyr: bool):
    """Boxes of occupied voxels with gaps between them, rays towards the
    middle, and proposals whose far end falls on each ray's third sample."""
    rng = np.random.default_rng(11)
    fine = np.zeros((128, 128, 128), np.uint8)
    for _ in range(60):
        c = rng.integers(16, 112, size=3)
        h = rng.integers(2, 7, size=3)
        fine[c[2] - h[2]:c[2] + h[2], c[1] - h[1]:c[1] + h[1], c[0] - h[0]:c[0] + h[0]] = 1
    levels = pyramid.build_pyramid(fine, 3)
    occ = levels[1]
    sc, _ = scene_and_dist("tiny")
    tables = sc.tables.copy()
    tables[:, :, 0] -= 1.5                                # thinner: rays go on past their third sample
    inp = OracleInputs(tables=tables, occ=occ, dist=distance_grid_edt(occ), mlp=sc.mlp,
                       resolutions=sc.cfg.resolutions, domain=CONTRACT, roi_half=2.0,
                       step=float(synth.CONTRACT_STEP), max_samples=1024, t_threshold=1e-4,
                       pyramid=levels if pyr else None, use_dist=True)
    n = 350
    o = rng.uniform(-3, 3, size=(n, 3)).astype(F32)
    dd = rng.uniform(-1.2, 1.2, size=(n, 3)) - o
    d = (dd / np.linalg.norm(dd, axis=1, keepdims=True)).astype(F32)
    plain = render(inp, o, d)
    starts = np.r_[0, np.cumsum(plain.n_samples)[:-1]]
    near, far = np.full(n, 0.5, F32), np.full(n, 1.0, F32)
    some = plain.n_samples > 4
    near[some] = plain.s_t[starts[some] + 1]              # use_near skips the first sample
    far[some] = plain.s_t[starts[some] + 2]
    conf = (rng.uniform(size=n) < 0.9).astype(F32)
    prop = np.stack([near, far, far, conf], axis=1).astype(F32)
    return sc, inp, fine, o, d, prop


@pytest.mark.parametrize("use_near", [False, True])
@pytest.mark.parametrize("pyr", [False, True])
def test_resumed_rays_match_oracle(pyr, use_near):
    import torch
    from paper_2407_10482_amd.renderer import Renderer
    print(f"[far guard, contracted, pyramid {pyr}, near {use_near}]", flush=True)
    sc, inp, fine, o, d, prop = _scene(pyr)
    n = len(o)
    margin = 0.25 * inp.step
    res, fb = render_proposal(inp, o, d, prop, 0.5, margin, use_near=use_near, far_guard=GUARD)
    # rays that went on, and of those the ones whose very next lattice point is a sample
    hi = prop[:, 1] + F32(margin)
    past = (res.s_t > hi[res.s_ray]) & (prop[res.s_ray, 3] >= 0.5) & ~fb[res.s_ray]
    first = past & np.r_[False, ~past[:-1] & (res.s_ray[1:] == res.s_ray[:-1])]
    nxt = np.nonzero(first)[0]
    assert len(nxt) > 100 and (res.s_k[nxt] == res.s_k[nxt - 1] + 1).sum() > 50
    kw = dict(occ_levels=3, occ_fine_res=128) if pyr else {}
    r = Renderer(sc.cfg.resolutions, sc.cfg.log2_table, 0, CONTRACT, 2.0, 64, inp.step, 1024, 1e-4,
                 use_distance=True, **kw)
    r.load_tables(*to_gpu(inp.tables))
    r.load_mlp(*to_gpu(inp.mlp))
    (r.load_occupancy_pyramid if pyr else r.load_occupancy)(*to_gpu(fine if pyr else inp.occ))
    out = r.alloc_outputs(n, labels=True)
    out["dist_loss"] = torch.empty((n,), device="cuda")
    out["fallback"] = torch.empty((n,), dtype=torch.int32, device="cuda")
    go, gd, gp = to_gpu(o, d, prop)
    r.render_intervals(go, gd, gp, 0.5, margin, out=out, use_near=use_near, far_guard=GUARD)
    got = {k: v.cpu().numpy() for k, v in out.items()}
    assert np.array_equal(got["fallback"].astype(bool), fb)
    assert np.array_equal(got["n_samples"], res.n_samples)
    assert np.array_equal(got["n_reads"], res.n_reads)
    assert np.array_equal(got["t_final"].view(np.uint32), res.t_final32.view(np.uint32))
    assert np.abs(got["rgb"] - res.rgb).max() < 1e-5
    before = np.where(np.r_[True, res.s_ray[1:] != res.s_ray[:-1]], 1.0,
                      np.r_[1.0, res.extra["s_T"][:-1].astype(np.float64)])
    want, _ = ray_distortion(n, res.s_ray, res.s_k, before - res.extra["s_T"], inp.step)
    assert np.abs(got["dist_loss"] - want).max() <= 1e-5 * max(1.0, np.abs(want).max())
