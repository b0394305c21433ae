"""Timed cases of the render path: what a user of the library has it do.

A user renders frames (single previews up to batches of full-HD views, in
each table type, with the hash or the baked feature model), trains a scene
(forward, backward, Adam; the hash model, the baked one, with the
distortion regulariser or the view-dependent MLP), rebuilds the occupancy
structures when the scene's geometry changes, and trains the sample-interval
proposal.  The scenes are synthetic with the distributions of the
repository's own workloads (blob mixtures; random tables), drawn on the GPU
from a seed.

``prepare`` makes the inputs and the renderer, ``run`` is one pass through
the public entry points, ``exact`` the same outputs in float64 with plain
torch operations.
"""
import math

import numpy as np
import torch

from paper_2407_10482_amd.renderer import (Proposal, Renderer, adam_step, proposal_init, render_differentiable,
                                           render_differentiable_baked, render_differentiable_view)

F32, BF16, FP8 = 0, 1, 2
CONTRACT_STEP = float(np.float32(2.0 * math.sqrt(3.0) / 512.0))
BOX_STEP = 1.0 / 256.0
THRESHOLD = float(np.float32(1e-4))
MAX_SAMPLES = 1024
LR, BETA1, BETA2, EPS, ADAM_STEP = 1e-5, 0.9, 0.99, 1e-8, 1000
DIST_WEIGHT = 1e-3
PROP_MARGIN = 4.0 / 256.0


def _case(name, do, **kw):
    c = dict(name=name, do=do, model="hash", domain="box", levels=8, n_min=16, n_max=256, log2_table=14,
             dtype=F32, occ_res=64, pyramid=0, coarse_res=0, view_mlp=False, views=1, width=64, height=64,
             aux=False, regulariser=False, phase=1)
    c.update(kw)
    return c


HD = dict(domain="contract", levels=16, n_max=4096, log2_table=19, occ_res=256)


def listed():
    return [
        # the smallest call: a 64x64 preview with all per-ray outputs; latency counts
        _case("preview_64", "render", aux=True),
        # an ordinary interactive frame: 1200x800, float32 tables, all per-ray outputs
        _case("frame_f32_1200x800", "render", width=1200, height=800, aux=True, **HD),
        # one full-HD frame from bfloat16 tables
        _case("frame_bf16_1080p", "render", width=1920, height=1080, dtype=BF16, **HD),
        # an odd-sized window (waves straddle image edges) from FP8 tables
        _case("frame_fp8_1277x717", "render", width=1277, height=717, dtype=FP8, **HD),
        # the headline workload: eight full-HD views in one call
        _case("views8_f32_1080p", "render", views=8, width=1920, height=1080, **HD),
        # the paper's representation: baked coarse grid, two gated fine levels, pyramid march, view-dependent MLP
        _case("paper_1080p", "render", model="baked", domain="contract", levels=2, n_min=1024, log2_table=22,
              occ_res=256, pyramid=5, coarse_res=512, view_mlp=True, width=1920, height=1080),
        # training steps: 2^18 rays of 16 small views, small and large hash tables
        _case("train_8x2p14", "train", views=16, width=128, height=128),
        _case("train_16x2p19", "train", views=16, width=128, height=128, levels=16, n_max=4096, log2_table=19),
        # training the paper's representation, an odd ray count
        _case("train_baked_view", "train", model="baked", levels=2, n_min=128, pyramid=3, occ_res=64,
              coarse_res=64, view_mlp=True, views=5, width=117, height=113),
        # a small batch with the distortion regulariser: launches and serial depth count
        _case("train_reg_small", "train", width=67, height=61, regulariser=True),
        # the occupancy structures after a geometry update: 512^3 .. 32^3 pyramid and 256^3 distance grid
        _case("occupancy_pyramid_512", "occupancy", occ_res=256, pyramid=5),
        # one step of the proposal network on a batch of 2^14 rays
        _case("proposal_train_2p14", "proposal", width=128, height=128, phase=2),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges."""
    do = rng.choice(["render"] * 5 + ["train"] * 3 + ["occupancy", "proposal"])
    kw = {}
    if do in ("render", "train"):
        if rng.random() < 0.3:
            kw.update(model="baked", levels=rng.randint(1, 4), n_min=128, coarse_res=rng.randint(48, 160))
        else:
            kw.update(levels=rng.randint(4, 16), n_max=_log_int(rng, 128, 4096), log2_table=rng.randint(12, 19))
        if rng.random() < 0.3:
            kw.update(pyramid=3, occ_res=rng.choice([32, 64, 128]))
        kw.update(view_mlp=rng.random() < 0.25)
    if do == "render":
        kw.update(views=rng.randint(1, 3), width=_log_int(rng, 9, 1400), height=_log_int(rng, 9, 900),
                  dtype=rng.choice([F32, F32, BF16, FP8]), aux=rng.random() < 0.5)
        if rng.random() < 0.6:
            kw.update(domain="contract", occ_res=rng.choice([128, 256]) if "pyramid" not in kw else 128)
    elif do == "train":
        kw.update(views=rng.randint(1, 12), width=_log_int(rng, 24, 140), height=_log_int(rng, 24, 140),
                  regulariser=rng.random() < 0.3)
    elif do == "occupancy":
        if rng.random() < 0.5:
            kw.update(domain="contract", occ_res=rng.randint(32, 288))
        else:
            kw.update(domain="contract", occ_res=rng.choice([64, 128]), pyramid=3)
    else:
        kw.update(width=_log_int(rng, 8, 320), height=_log_int(rng, 8, 320), phase=rng.randint(1, 2))
    c = _case("", do, **kw)
    del c["name"]
    return c


# ---------------------------------------------------------------------------
# inputs: blob scenes, random tables, pinhole cameras

def _resolutions(c):
    L = c["levels"]
    if c["model"] == "baked":
        return [c["n_min"] << l for l in range(L)]
    b = (c["n_max"] / c["n_min"]) ** (1.0 / max(L - 1, 1))
    return [int(math.floor(c["n_min"] * b ** l + 1e-6)) for l in range(L)]


def _half(c):
    return 1.0 if c["domain"] == "box" else 2.0


def _step(c):
    return BOX_STEP if c["domain"] == "box" else CONTRACT_STEP


def _cameras(c, rng):
    n = c["views"]
    if c["domain"] == "box":
        v = rng.normal(size=(n, 3))
        return v / np.linalg.norm(v, axis=1, keepdims=True)
    th = 2.0 * np.pi * (np.arange(n) / n + rng.uniform())
    return np.stack([3.0 * np.cos(th), 3.0 * np.sin(th), np.zeros(n)], axis=1)


def _blobs(c, rng, cams):
    if c["domain"] == "box":
        return rng.uniform(-0.5, 0.5, size=(3, 3)), rng.uniform(0.1, 0.3, size=3)
    r = np.linalg.norm(cams, axis=1, keepdims=True)
    inside = cams / r * (2.0 - 1.0 / r)
    mu, sig = [], []
    while len(mu) < 200:
        p, s = rng.uniform(-1.9, 1.9, size=3), rng.uniform(0.03, 0.12)
        if np.linalg.norm(p) < 1.9 and np.min(np.linalg.norm(inside - p, axis=1)) > 3.0 * s:
            mu.append(p)
            sig.append(s)
    return np.array(mu), np.array(sig)


def _density(axis, mu, sig):
    """Blob mixture on the lattice axis^3 ([z, y, x]); each blob to 4 of its deviations."""
    n = len(axis)
    rho = torch.zeros((n, n, n), dtype=torch.float32, device="cuda")
    x = torch.from_numpy(axis).cuda()
    for m, s in zip(mu, sig):
        cut = [np.searchsorted(axis, [m[a] - 4 * s, m[a] + 4 * s]) for a in range(3)]
        if any(hi <= lo for lo, hi in cut):
            continue
        g = [torch.exp(-(x[lo:hi] - m[a]) ** 2 / (2 * s * s)).float() for a, (lo, hi) in enumerate(cut)]
        rho[cut[2][0]:cut[2][1], cut[1][0]:cut[1][1], cut[0][0]:cut[0][1]] += (
            g[2][:, None, None] * g[1][None, :, None] * g[0][None, None, :])
    return rho


def _rays(c, cams):
    """Pinhole rays (60 degrees across), view after view, in 8x8-pixel tiles."""
    W, H = c["width"], c["height"]
    row, col = np.divmod(np.arange(W * H), W)
    order = np.lexsort((col % 8, row % 8, col // 8, row // 8))
    row, col = (torch.from_numpy(v[order]).cuda() for v in (row, col))
    tan = math.tan(math.radians(30.0))
    xn = (2.0 * (col + 0.5) / W - 1.0) * tan
    yn = (1.0 - 2.0 * (row + 0.5) / H) * tan * H / W
    os_, ds = [], []
    for p in cams:
        fwd = -p / np.linalg.norm(p)
        up = np.array([0.0, 0.0, 1.0]) if abs(fwd[2]) < 0.999 else np.array([0.0, 1.0, 0.0])
        right = np.cross(fwd, up)
        right /= np.linalg.norm(right)
        up = np.cross(right, fwd)
        f, r, u = (torch.from_numpy(v).cuda() for v in (fwd, right, up))
        d = f + xn.double()[:, None] * r + yn.double()[:, None] * u
        ds.append((d / d.norm(dim=1, keepdim=True)).float())
        os_.append(torch.from_numpy(p).cuda().float().expand(W * H, 3))
    return torch.cat(os_).contiguous(), torch.cat(ds).contiguous()


def _mlp(c, g):
    dims = (23, 64, 64, 3) if c["view_mlp"] else (7, 16, 16, 3)
    parts = []
    for fin, fout in zip(dims, dims[1:]):
        a = math.sqrt(6.0 / (fin + fout))
        parts += [(torch.rand(fout * fin, generator=g, device="cuda") * 2 - 1) * a,
                  torch.zeros(fout, device="cuda")]
    return torch.cat(parts).contiguous()


def _inputs(c, seed):
    """Everything the case's program holds before its call, from the seed alone."""
    rng = np.random.default_rng([seed, 77])
    g = torch.Generator(device="cuda").manual_seed(seed)
    cams = _cameras(c, rng)
    mu, sig = _blobs(c, rng, cams)
    h = _half(c)
    R = c["occ_res"] if not c["pyramid"] else _fine_res(c)
    s = {"occ": (_density(-h + (np.arange(R) + 0.5) * (2 * h / R), mu, sig) > 0.01).to(torch.uint8)}
    if c["do"] == "occupancy":
        return s
    s["o"], s["d"] = _rays(c, cams)
    n, L, T = len(s["o"]), c["levels"], 1 << c["log2_table"]
    tab = torch.empty((L, T, 9), device="cuda")
    s["mlp"] = _mlp(c, g)
    if c["model"] == "hash":
        scale = 600.0 if c["domain"] == "box" else 400.0
        z2 = torch.randn((L, T, 3), generator=g, device="cuda").square().sum(2)
        tab[:, :, 0] = torch.log(scale * torch.exp(-0.5 * z2) + 1e-4)
        tab[:, :, 1:4] = torch.rand((L, T, 3), generator=g, device="cuda")
        tab[:, :, 4:] = 0.5 * torch.randn((L, T, 5), generator=g, device="cuda")
    else:
        std = torch.tensor([0.5] + [0.2] * 3 + [0.5] * 4 + [0.0], device="cuda")
        tab.copy_(torch.randn((L, T, 9), generator=g, device="cuda") * std)
        nb = (c["coarse_res"] + 8) // 8
        rho = _density(-h + np.arange(8 * nb) * (2 * h / c["coarse_res"]), mu, sig)
        rho = rho.view(nb, 8, nb, 8, nb, 8).permute(0, 2, 4, 1, 3, 5).reshape(nb ** 3, 512)
        keep = rho.amax(1).topk(nb ** 3 // 3).indices.sort().values     # the densest third is stored
        index = torch.full((nb ** 3,), -1, dtype=torch.int32, device="cuda")
        index[keep] = torch.arange(len(keep), dtype=torch.int32, device="cuda")
        scale = 1e4 if c["domain"] == "box" else 4000.0
        atlas = torch.randn((len(keep), 512, 8 + 2 * L), generator=g, device="cuda")
        atlas[:, :, 0] = torch.log(scale * rho[keep] + 1e-4)
        atlas[:, :, 1:4] = torch.rand((len(keep), 512, 3), generator=g, device="cuda")
        atlas[:, :, 4:8] *= 0.5
        s["index"] = index.view(nb, nb, nb)
        s["atlas"] = atlas.view(len(keep), 8, 8, 8, 8 + 2 * L)
        s["default"] = [math.log(1e-4)] + [0.0] * (7 + 2 * L)
    s["tables"] = tab
    if c["do"] == "train":
        s["target"] = torch.rand((n, 3), generator=g, device="cuda")
        names = [k for k in ("tables", "atlas", "mlp") if k in s]
        # moments of a step in mid-training: m around the gradients' size, v around its square
        s["m"] = {k: torch.randn(s[k].shape, generator=g, device="cuda") * 1e-7 for k in names}
        s["v"] = {k: (torch.rand(s[k].shape, generator=g, device="cuda") + 0.5) * 1e-12 for k in names}
    if c["do"] == "proposal":
        near = torch.rand(n, generator=g, device="cuda")
        far = near + torch.rand(n, generator=g, device="cuda")
        s["labels"] = torch.stack([near, far, 0.5 * (near + far),
                                   (torch.rand(n, generator=g, device="cuda") < 0.8).float()], 1).contiguous()
        s["net"] = proposal_init(seed)
        s["m"] = torch.randn(s["net"].shape, generator=g, device="cuda") * 1e-3
        s["v"] = (torch.rand(s["net"].shape, generator=g, device="cuda") + 0.5) * 1e-4
    return s


def _fine_res(c):
    """The finest pyramid level: two resolutions of the distance grid, one above it (at least 32 at the coarsest)."""
    return max(2 * c["occ_res"], 32 << (c["pyramid"] - 1))


# ---------------------------------------------------------------------------
# the cases' programs

def prepare(case, seed):
    c = case
    s = _inputs(c, seed)
    r = Renderer(_resolutions(c), c["log2_table"], c["dtype"], 0 if c["domain"] == "box" else 1, _half(c),
                 c["occ_res"], _step(c), MAX_SAMPLES, 1e-4, feature_model=int(c["model"] == "baked"),
                 coarse_res=c["coarse_res"], occ_levels=c["pyramid"],
                 occ_fine_res=_fine_res(c) if c["pyramid"] else 0, use_distance=True,
                 mlp_dims=(23, 64, 64, 3) if c["view_mlp"] else (7, 16, 16, 3))
    s.update(case=c, r=r)
    if c["do"] == "occupancy":
        return s
    if c["do"] == "proposal":
        s["net"] = Proposal(s["net"], r)
        s["net"].m.copy_(s.pop("m"))
        s["net"].v.copy_(s.pop("v"))
        s["net"].step = ADAM_STEP
        s["loss"] = torch.zeros((1,), device="cuda")
        return s
    (r.load_occupancy_pyramid if c["pyramid"] else r.load_occupancy)(s["occ"])
    r.load_tables(s["tables"])
    r.load_mlp(s["mlp"])
    if c["model"] == "baked":
        r.load_coarse(s["index"], s["atlas"], s["default"])
    if c["do"] == "render":
        n = len(s["o"])
        s["out"] = r.alloc_outputs(n) if c["aux"] else {"rgb": torch.empty((n, 3), device="cuda")}
    else:
        s["params"] = {k: s[k].requires_grad_(True) for k in s["m"]}
        s["step"] = ADAM_STEP
    return s


def run(state):
    s, c = state, state["case"]
    r = s["r"]
    if c["do"] == "render":
        return r.render(s["o"], s["d"], out=s["out"])
    if c["do"] == "occupancy":
        (r.load_occupancy_pyramid if c["pyramid"] else r.load_occupancy)(s["occ"])
        return r.export_distance()
    if c["do"] == "proposal":
        s["loss"].zero_()
        s["net"].train_step(s["o"], s["d"], s["labels"], LR, phase=c["phase"], margin=PROP_MARGIN, loss=s["loss"])
        return {"params": s["net"].params, "m": s["net"].m, "v": s["net"].v, "loss": s["loss"]}
    p = s["params"]
    for q in p.values():
        q.grad = None
    args = (s["o"], s["d"])
    if c["view_mlp"]:
        got = render_differentiable_view(r, p["tables"], p["mlp"], *args, atlas=p.get("atlas"),
                                         with_dist=c["regulariser"])
    elif c["model"] == "baked":
        got = render_differentiable_baked(r, p["tables"], p["atlas"], p["mlp"], *args, with_dist=c["regulariser"])
    else:
        got = render_differentiable(r, p["tables"], p["mlp"], *args, with_dist=c["regulariser"])
    rgb, dist = got if c["regulariser"] else (got, None)
    loss = torch.mean((rgb - s["target"]) ** 2)
    if dist is not None:
        loss = loss + DIST_WEIGHT * torch.mean(dist)
    loss.backward()
    s["step"] += 1
    with torch.no_grad():
        for k, q in p.items():
            adam_step(q, q.grad, s["m"][k], s["v"][k], s["step"], LR, BETA1, BETA2, EPS)
    return {"rgb": rgb, "grad": {k: q.grad for k, q in p.items()}, "params": dict(p)}


# ---------------------------------------------------------------------------
# what a pass cannot do without

def work(case):
    c = case
    if c["do"] == "occupancy":
        R = c["occ_res"]
        cells = _fine_res(c) ** 3 if c["pyramid"] else R ** 3
        # the occupancy in, the distance grid out as the march reads it and as exported; a distance per voxel and axis
        return {"bytes": cells + 3 * R ** 3, "flops": 3 * R ** 3}
    n = c["views"] * c["width"] * c["height"]
    if c["do"] == "proposal":
        macs = 48 * 64 + 64 * 64 + 64 * 4
        return {"bytes": n * 40 + 7556 * 4 * 6, "flops": 6 * macs * n}
    L, T = c["levels"], 1 << c["log2_table"]
    samples = 15 * n            # evaluated samples of these scenes, about 15 to 18 a ray
    entry = {F32: 36, BF16: 18, FP8: 9}[c["dtype"]]
    tables = min(L * T, samples * L * 8) * entry
    macs = L * (8 * (9 if c["model"] == "hash" else 8) + 8)
    params = L * T * 9
    if c["model"] == "baked":
        C = 8 + 2 * L
        verts = min((c["coarse_res"] + 1) ** 3 // 3, samples * 8)     # stored vertices: about a third
        tables += verts * C * 4
        macs += 8 * C
        params += verts * C
    ray_macs = 5700 if c["view_mlp"] else 416
    flops = 2 * (samples * macs + n * ray_macs)
    io = n * (24 + 12 + (44 if c["aux"] else 0))
    if c["do"] == "render":
        return {"bytes": io + tables, "flops": flops}
    # training: forward and backward read the tables, the gradient is written, Adam reads 4 and writes 3 floats
    return {"bytes": io + 2 * tables + params * 4 * 8, "flops": 3 * flops + 12 * params}


# ---------------------------------------------------------------------------
# the same outputs in float64

def _stored(c, tab):
    """The tables as the storage type holds them, float64."""
    if c["dtype"] == BF16:
        return tab.bfloat16().double()
    if c["dtype"] == FP8:
        amax = tab.abs().amax(1, keepdim=True)
        sc = torch.where(amax > 0, amax / 448.0, torch.ones_like(amax))
        return (tab / sc).to(torch.float8_e4m3fn).double() * sc.double()
    return tab.double()


_BITS = [[k & 1, (k >> 1) & 1, (k >> 2) & 1] for k in range(8)]


def _cells(u, N):
    """u [B, 3] on lattices of resolution N [L]: corners [B, L, 8, 3] and weights [B, L, 8]."""
    bits = torch.tensor(_BITS, device="cuda")
    p = u[:, None, :] * N[None, :, None].double()
    i = torch.minimum(p.floor().clamp(min=0).long(), N[None, :, None] - 1)
    f = (p - i)[:, :, None, :]
    w = torch.where(bits.bool(), f, 1.0 - f).prod(3)
    return i[:, :, None, :] + bits, w


def _features(c, s, u):
    """The fused deferred feature [B, 8] at grid coordinates u in [0, 1]^3."""
    L, T = c["levels"], 1 << c["log2_table"]
    q, w = _cells(u, torch.tensor(_resolutions(c), device="cuda"))
    m = 0xFFFFFFFF
    idx = (q[..., 0] ^ ((q[..., 1] * 2654435761) & m) ^ ((q[..., 2] * 805459861) & m)) & (T - 1)
    idx = idx + (torch.arange(L, device="cuda") * T)[None, :, None]
    v = (s["tab64"].view(L * T, 9)[idx] * w[..., None]).sum(2)
    if c["model"] == "hash":
        return (torch.softmax(v[..., 8], 1)[..., None] * v[..., :8]).sum(1)
    q, w = _cells(u, torch.tensor([c["coarse_res"]], device="cuda"))
    q, w = q[:, 0], w[:, 0]
    b = q >> 3
    bid = s["index"][b[..., 2], b[..., 1], b[..., 0]].long()
    loc = ((q[..., 2] & 7) * 8 + (q[..., 1] & 7)) * 8 + (q[..., 0] & 7)
    atlas = s["atlas64"].view(-1, 8 + 2 * L)
    row = atlas[(bid.clamp(min=0) * 512 + loc)]
    dflt = torch.tensor(np.float32(s["default"]), device="cuda").double()
    co = (torch.where((bid >= 0)[..., None], row, dflt) * w[..., None]).sum(1)
    gate = torch.sigmoid(co[:, 8:]).view(-1, L, 2)
    return torch.cat([co[:, :1] + (gate[..., :1] * v[..., :1]).sum(1),
                      co[:, 1:8] + (gate[..., 1:] * v[..., 1:8]).sum(1)], 1)


def _walk(c, occ, o, d, alive, visit):
    """March every lattice point; visit(rays, u, t, k) for those in occupied voxels (it clears alive)."""
    h, step, R = _half(c), _step(c), occ.shape[0]
    o, d = o.double(), d.double()
    t = torch.zeros(len(o), dtype=torch.float64, device="cuda")
    t1 = torch.full_like(t, math.inf)
    if c["domain"] == "box":
        a, b = (-h - o) / d, (h - o) / d
        t = torch.minimum(a, b).amax(1).clamp(min=0)
        t1 = torch.maximum(a, b).amin(1)
    t0 = t.clone()
    dn2 = (d * d).sum(1)
    for k in range(1 << 16):
        if k % 8 == 0:
            live = alive.nonzero()[:, 0]
            if not len(live):
                break
            lo, ld, ln2 = o[live], d[live], dn2[live]
        tc = t0[live] + k * step if c["domain"] == "box" else t[live]
        x = lo + tc[:, None] * ld
        ok = alive[live] & (tc < t1[live])
        if c["domain"] == "contract":
            r = x.norm(dim=1)
            out = r > 1.0
            inv = 1.0 / r.clamp(min=1.0)
            sc = (2.0 - inv) * inv
            xd = (x * ld).sum(1) * inv
            ok = ok & ~(out & (inv < step) & (xd >= 0))
            jn = torch.where(out, (sc * sc * (ln2 - xd * xd).clamp(min=0) + (xd * inv * inv) ** 2).sqrt(), ln2.sqrt())
            x = torch.where(out[:, None], sc[:, None] * x, x)
            t[live] = tc + step / jn
        alive[live] = ok
        u = (x + h) / (2 * h)
        q = (u * R).floor().clamp(0, R - 1).long()
        hit = ok & (occ[q[:, 2], q[:, 1], q[:, 0]] != 0)
        at = hit.nonzero()[:, 0]
        if len(at):
            visit(live[at], u[at], tc[at], k)


def _sh(d):
    x, y, z = (d.double() / d.double().norm(dim=1, keepdim=True)).unbind(1)
    p = math.pi
    a, b = math.sqrt(15 / p) / 2, math.sqrt(35 / (2 * p)) / 4
    e, q, g = math.sqrt(21 / (2 * p)) / 4, math.sqrt(105 / p), math.sqrt(3 / (4 * p))
    return torch.stack([torch.full_like(x, 0.5 / math.sqrt(p)), g * y, g * z, g * x,
                        a * x * y, a * y * z, math.sqrt(5 / p) / 4 * (3 * z * z - 1), a * x * z,
                        a / 2 * (x * x - y * y), b * y * (3 * x * x - y * y), q / 2 * x * y * z,
                        e * y * (5 * z * z - 1), math.sqrt(7 / p) / 4 * z * (5 * z * z - 3),
                        e * x * (5 * z * z - 1), q / 4 * z * (x * x - y * y), b * x * (x * x - 3 * y * y)], 1)


def _colour(c, mlp, cd, fv, d):
    x = torch.cat([cd, fv] + ([_sh(d)] if c["view_mlp"] else []), 1)
    dims = (23, 64, 64, 3) if c["view_mlp"] else (7, 16, 16, 3)
    at = 0
    for j, (i, n) in enumerate(zip(dims, dims[1:])):
        W, b = mlp[at:at + i * n].view(n, i), mlp[at + i * n:at + i * n + n]
        at += i * n + n
        x = x @ W.T + b
        x = torch.relu(x) if j < 2 else x
    return torch.sigmoid(cd + x)


def _march64(c, s, o, d, keep):
    """Composite every ray; with keep also its sample list (ray, slot, u, k)."""
    n, step = len(o), _step(c)
    z = lambda *shape: torch.zeros(shape, dtype=torch.float64, device="cuda")  # noqa: E731
    T, cd, fv, depth = z(n) + 1.0, z(n, 3), z(n, 4), z(n)
    ns = torch.zeros(n, dtype=torch.long, device="cuda")
    alive = torch.ones(n, dtype=torch.bool, device="cuda")
    kept = []

    def visit(rays, u, t, k):
        f = torch.cat([_features(c, s, part) for part in u.split(1 << 18)])
        e = torch.exp(-torch.exp(f[:, 0]) * step)
        w = T[rays] * (1.0 - e)
        cd[rays] += w[:, None] * f[:, 1:4]
        fv[rays] += w[:, None] * f[:, 4:]
        depth[rays] += w * t
        T[rays] *= e
        if keep:
            kept.append((rays, ns[rays], u, torch.full_like(rays, k)))
        ns[rays] += 1
        alive[rays] &= (T[rays] >= THRESHOLD) & (ns[rays] < MAX_SAMPLES)

    with torch.no_grad():
        _walk(c, s["occ"], o, d, alive, visit)
    return T, cd, fv, depth, kept


def _exact_train(c, s):
    names = list(s["m"])
    n, step = len(s["o"]), _step(c)
    leaf = {k: s[k].double().requires_grad_(True) for k in names}
    grad = {k: torch.zeros_like(leaf[k]) for k in names}
    with torch.no_grad():
        s["tab64"], s["atlas64"] = leaf["tables"].detach(), leaf.get("atlas", leaf["mlp"]).detach()
        kept = _march64(c, s, s["o"], s["d"], True)[4]
    empty = torch.zeros(0, dtype=torch.long, device="cuda")
    ray, slot, u, k = (torch.cat(v) for v in zip(*kept)) if kept else (empty, empty, empty.double().view(0, 3), empty)
    order = torch.argsort(ray, stable=True)
    ray, slot, u, k = ray[order], slot[order], u[order], k[order]
    s["tab64"], s["atlas64"] = leaf["tables"], leaf.get("atlas")
    rgbs, size = [], 1 << 14
    for lo in range(0, n, size):
        m = min(size, n - lo)
        a, b = torch.searchsorted(ray, torch.tensor([lo, lo + m], device="cuda")).tolist()
        rr, ss = ray[a:b] - lo, slot[a:b]
        S = int(ss.max()) + 1 if b > a else 1
        cd = torch.zeros((m, 3), dtype=torch.float64, device="cuda")
        fv = torch.zeros((m, 4), dtype=torch.float64, device="cuda")
        dist = torch.zeros((), dtype=torch.float64, device="cuda")
        if b > a:
            f = _features(c, s, u[a:b])
            grid = torch.zeros((m, S), dtype=torch.float64, device="cuda")
            tau = grid.index_put((rr, ss), torch.exp(f[:, 0]) * step)
            W = torch.exp(-(tau.cumsum(1) - tau)) * (1.0 - torch.exp(-tau))
            w = W[rr, ss][:, None]
            cd = cd.index_add(0, rr, w * f[:, 1:4])
            fv = fv.index_add(0, rr, w * f[:, 4:])
            if c["regulariser"]:
                mid = grid.index_put((rr, ss), (k[a:b].double() + 0.5) * step)
                Wm = W * mid
                dist = (2 * W * (mid * (W.cumsum(1) - W) - (Wm.cumsum(1) - Wm)) + step / 3 * W * W).sum()
        rgb = _colour(c, leaf["mlp"], cd, fv, s["d"][lo:lo + m])
        loss = ((rgb - s["target"][lo:lo + m].double()) ** 2).sum() / (3 * n) + DIST_WEIGHT * dist / n
        for key, gr in zip(names, torch.autograd.grad(loss, [leaf[q] for q in names], allow_unused=True)):
            if gr is not None:
                grad[key] += gr
        rgbs.append(rgb.detach())
        del loss, rgb
    params, c1, c2 = {}, 1 - BETA1 ** (ADAM_STEP + 1), 1 - BETA2 ** (ADAM_STEP + 1)
    for key in names:
        m1 = BETA1 * s["m"][key].double() + (1 - BETA1) * grad[key]
        v1 = BETA2 * s["v"][key].double() + (1 - BETA2) * grad[key] ** 2
        params[key] = leaf[key].detach() - LR * (m1 / c1) / ((v1 / c2).sqrt() + EPS)
    return {"rgb": torch.cat(rgbs), "grad": grad, "params": params}


def _exact_proposal(c, s):
    o, d, y, n = s["o"].double(), s["d"].double(), s["labels"].double(), len(s["o"])
    p = s["net"].double().requires_grad_(True)
    a = math.pi * torch.cat([o, d], 1)[:, :, None] * torch.tensor([1.0, 2.0, 4.0, 8.0], device="cuda").double()
    x = torch.stack([a.sin(), a.cos()], 3).reshape(n, 48)
    at = 0
    for i, w in ((48, 64), (64, 64), (64, 4)):
        x = x @ p[at:at + i * w].view(w, i).T + p[at + i * w:at + i * w + w]
        at += i * w + w
        x = torch.relu(x) if w == 64 else x
    valid = y[:, 3]
    r0, r1 = y[:, 0] - x[:, 0], y[:, 1] - x[:, 1]
    loss = (valid * (torch.maximum(0.05 * r0, -0.95 * r0) + torch.maximum(0.95 * r1, -0.05 * r1)
                     + (x[:, 2] - y[:, 2]) ** 2)).sum()
    if c["phase"] == 2:
        tgt = valid * ((x[:, 0] - PROP_MARGIN <= y[:, 0]) & (x[:, 1] + PROP_MARGIN >= y[:, 1])).double()
        sg = torch.sigmoid(x[:, 3])
        loss = loss - (tgt.detach() * torch.log(sg + 1e-12) + (1 - tgt.detach()) * torch.log(1 - sg + 1e-12)).sum()
    loss = loss / n
    g, = torch.autograd.grad(loss, p)
    m1, v1 = BETA1 * s["m"].double() + (1 - BETA1) * g, BETA2 * s["v"].double() + (1 - BETA2) * g * g
    c1, c2 = 1 - BETA1 ** (ADAM_STEP + 1), 1 - BETA2 ** (ADAM_STEP + 1)
    q = p.detach() - LR * (m1 / c1) / ((v1 / c2).sqrt() + EPS)
    return {"params": q, "m": m1, "v": v1, "loss": loss.detach().view(1)}


def exact(case, seed):
    c = case
    if c["do"] == "occupancy" or c["views"] * c["width"] * c["height"] > 3 << 20:
        return None                      # whole numbers, or too long
    s = _inputs(c, seed)
    if c["do"] == "proposal":
        return _exact_proposal(c, s)
    if c["do"] == "train":
        return _exact_train(c, s)
    s["tab64"] = _stored(c, s["tables"])
    if "atlas" in s:
        s["atlas64"] = s["atlas"].double()
    parts = []
    for lo in range(0, len(s["o"]), 1 << 20):
        o, d = s["o"][lo:lo + (1 << 20)], s["d"][lo:lo + (1 << 20)]
        T, cd, fv, depth, _ = _march64(c, s, o, d, False)
        parts.append((_colour(c, s["mlp"].double(), cd, fv, d), cd, fv, T, depth))
    rgb, cd, fv, T, depth = (torch.cat(v) for v in zip(*parts))
    out = {"rgb": rgb}
    if c["aux"] or c["view_mlp"]:
        out.update(c_d=cd, feat=fv)
    if c["aux"]:
        out.update(t_final=T, depth=depth, n_samples=None, n_reads=None)
    return out
