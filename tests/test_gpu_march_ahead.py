"""The march that runs ahead of the evaluation (the per-lane sample ring):
slabs of occupied voxels with gaps between them and unordered rays, so the
lanes of a wave meet their gaps at different samples and fill their rings to
different depths.  Sample lists, counts and read counts against the oracle,
with sample caps around the ring's depth (8)."""
import dataclasses

import numpy as np
import pytest

import synth
from helpers import to_gpu
from oracle.distgrid import distance_grid_edt
from oracle.render import inputs_from_scene, render

pytestmark = pytest.mark.gpu


def _slab_scene(domain: str, max_samples: int):
    cfg = synth.tiny()
    cfg.max_samples, cfg.density_scale, cfg.log2_table = max_samples, 4.0, 10
    if domain == "contract":
        cfg.domain, cfg.roi_half, cfg.step = synth.configs.DOMAIN_CONTRACT, 2.0, 16 * synth.configs.CONTRACT_STEP
        cfg.occ_res = 48
    else:
        cfg.step = 1.0 / 32.0
    sc = synth.make_scene(dataclasses.replace(cfg, domain=synth.configs.DOMAIN_BOX))
    R = cfg.occ_res
    z = np.arange(R)
    occ = np.zeros((R, R, R), np.uint8)
    occ[(z % 11) < 2] = 1                    # thin slabs, 9 voxels apart
    occ[:, :, R // 2:][:, (z % 7) == 3] = 1  # and denser sheets in one half
    return dataclasses.replace(sc, cfg=cfg, occ=occ)


@pytest.mark.parametrize("max_samples", [1, 7, 8, 9, 1024])
@pytest.mark.parametrize("domain", ["box", "contract"])
def test_samples_found_ahead(domain, max_samples):
    print(f"[march ahead {domain} cap {max_samples}]", flush=True)
    from paper_2407_10482_amd.renderer import Renderer
    sc = _slab_scene(domain, max_samples)
    cfg = sc.cfg
    inp = inputs_from_scene(sc, distance_grid_edt(sc.occ), 0)
    rng = np.random.default_rng(3)
    n = 333
    o = rng.uniform(-1.2, 1.2, size=(n, 3)).astype(np.float32)
    d = rng.normal(size=(n, 3)).astype(np.float32)
    d[5] = np.nan                            # an empty ray among them
    r = Renderer.from_config(cfg)
    r.load_scene(*to_gpu(sc.tables, sc.occ, sc.mlp))
    go, gd = to_gpu(o, d)
    ref = render(inp, o, d)
    if max_samples == 1024:                  # gaps at different samples, rays deeper than the ring
        assert ref.n_samples.max() > 16
    cap = 64
    sk, ns, nr = (x.cpu().numpy() for x in r.march(go, gd, cap=cap))
    assert np.array_equal(ns, ref.n_samples) and np.array_equal(nr, ref.n_reads)
    starts = np.r_[0, np.cumsum(ref.n_samples)[:-1]]
    for i in range(n):
        m = min(int(ref.n_samples[i]), cap)
        assert np.array_equal(sk[i, :m], ref.s_k[starts[i]:starts[i] + m]) and (sk[i, m:] == -1).all()
    for labels in (False, True):             # the plain kernel and the one with label outputs
        out = r.render(go, gd, out=r.alloc_outputs(n, labels=labels))
        assert np.array_equal(out["n_samples"].cpu().numpy(), ref.n_samples)
        assert np.array_equal(out["n_reads"].cpu().numpy(), ref.n_reads)
        assert np.abs(out["rgb"].cpu().numpy() - ref.rgb).max() < 1e-5


# 81,920 rays and fewer take sixteen lanes a ray, more take the ring: the same
# bits either way, so each side checks the other (and the oracle checks the
# small one above and in the parity tests)
@pytest.mark.parametrize("name,dtype", [("tiny", 0), ("tiny", 1), ("tiny", 2), ("tiny_pyramid", 0), ("baked_tiny", 0),
                                        ("baked_tiny_l3", 1), ("paper_tiny", 0), ("baked_tiny_sum", 0)])
def test_small_launches_match_large_ones(name, dtype):
    import torch
    from helpers import gpu_renderer, scene_and_dist
    print(f"[small launches {name} {dtype}]", flush=True)
    cfg = scene_and_dist(name, dtype)[0].cfg
    cams = synth.random_sphere_cameras(21, 1.0, seed=77)
    o, d, _ = synth.scene_rays(cfg, cams=cams, width=64, height=64)
    o, d = to_gpu(o[:81921], d[:81921])
    d[11] = float("nan")
    r = gpu_renderer(name, dtype)

    def render(n, labels):
        out = r.alloc_outputs(n, labels=labels)
        if labels:
            out["dist_loss"] = torch.empty((n,), device="cuda")
        return r.render(o[:n].contiguous(), d[:n].contiguous(), out=out)
    for labels in (False, True):
        want = render(81921, labels)
        assert int(want["n_samples"].max()) > 16          # rays of more than one round of sixteen
        for n in (1, 15, 16, 17, 4099, 81920):
            got = render(n, labels)
            for k, v in got.items():
                assert torch.equal(v.view(torch.int32), want[k][:n].contiguous().view(torch.int32)), (n, labels, k)


@pytest.mark.parametrize("domain", ["box", "contract"])
def test_ring_on_slabs(domain):
    """The slab scene's gaps through the one-lane kernel (a launch above the
    small ones), against the small launch of the same rays."""
    import torch
    from paper_2407_10482_amd.renderer import Renderer
    print(f"[ring on slabs {domain}]", flush=True)
    for cap in (7, 8, 9, 1024):
        sc = _slab_scene(domain, cap)
        rng = np.random.default_rng(5)
        n = 82000
        o, d = to_gpu(rng.uniform(-1.2, 1.2, size=(n, 3)).astype(np.float32),
                      rng.normal(size=(n, 3)).astype(np.float32))
        r = Renderer.from_config(sc.cfg)
        r.load_scene(*to_gpu(sc.tables, sc.occ, sc.mlp))
        whole = r.render(o, d)
        part = r.render(o[:4000].contiguous(), d[:4000].contiguous())
        for k, v in part.items():
            assert torch.equal(v.view(torch.int32), whole[k][:4000].contiguous().view(torch.int32)), (cap, k)
