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


# batches that pad the tables' rows (2^14 a level: from 3,276 rays on, baked from 8,192)
@pytest.mark.parametrize("name,n", [("tiny", 3276), ("tiny", 16500), ("baked_tiny", 8192), ("baked_tiny", 16500)])
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


@pytest.mark.parametrize("name,n", [("tiny", 3275), ("tiny", 3276), ("baked_tiny", 8191), ("baked_tiny", 8192)])
def test_around_the_rule(name, n):
    """Either side of the line from which rows are padded, against the batch in
    parts below it."""
    print(f"[padded rows around the rule {name} {n}]", flush=True)
    o, d, g = _rays(name, n)
    r = gpu_renderer(name)
    whole = _grads(r, o, d, g)
    parts = [_grads(r, *(x[lo:hi].contiguous() for x in (o, d, g))) for lo, hi in ((0, 40), (40, 3000), (3000, n))]
    for k, a in enumerate(whole):
        b = parts[0][k] + parts[1][k] + parts[2][k]
        assert float(b.abs().max()) > 0 and _close(a, b)


def test_padded_rows_hold_at_most_one_gib():
    """A baked scene whose tables (4 x 2^22) take 1 GiB of padded rows, and whose
    atlas (2^15 blocks) would take as much."""
    import torch
    from paper_2407_10482_amd.renderer import Renderer
    print("[padded rows: memory held]", flush=True)
    blocks = 1 << 15
    r = Renderer([256, 512, 1024, 2048], 22, occ_res=32, feature_model=1, coarse_res=255)
    r.load_tables(torch.zeros((4, 1 << 22, 9), device="cuda"))
    r.load_occupancy(torch.ones((32, 32, 32), dtype=torch.uint8, device="cuda"))
    r.load_mlp(torch.zeros((451,), device="cuda"))
    index = torch.arange(blocks, dtype=torch.int32, device="cuda").view(32, 32, 32)
    r.load_coarse(index, torch.zeros((blocks, 8, 8, 8, 16), device="cuda"), [0.0] * 16)
    n = 1 << 21                                           # T / 2: the tables' rows are padded
    o, g = torch.zeros((n, 3), device="cuda"), torch.ones((n, 3), device="cuda")
    d = torch.zeros((n, 3), device="cuda")                # rays without a direction: no samples
    grads = [torch.zeros(s, device="cuda") for s in ((4, 1 << 22, 9), (blocks, 8, 8, 8, 16), (451,))]
    r.backward_baked(o[:64], d[:64], g[:64], *grads)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    r.backward_baked(o, d, g, *grads)
    torch.cuda.synchronize()
    held = before - torch.cuda.mem_get_info()[0]
    # the rows, 59 MB of partials, and the allocator's rounding
    assert (1 << 30) <= held <= (1 << 30) + (128 << 20), held
    assert float(grads[0].abs().max()) == 0.0 and float(grads[1].abs().max()) == 0.0


def test_two_contexts_add_to_one_gradient():
    """Contexts on two streams accumulate into one table gradient: every
    addition to it is atomic, the padded rows' too."""
    import torch
    print("[padded rows: two contexts, one gradient]", flush=True)
    n, times = 16500, 24
    o, d, g = _rays("tiny", n)
    cf = torch.cat([g, g[:, :1].expand(n, 4)], 1).contiguous()
    rs = [gpu_renderer("tiny"), gpu_renderer("tiny")]
    one = torch.zeros((rs[0].L, rs[0].T, 9), device="cuda")
    rs[0].backward_features(o, d, cf, one)
    both = torch.zeros_like(one)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for _ in range(times):
        for r, s in zip(rs, streams):
            with torch.cuda.stream(s):
                r.backward_features(o, d, cf, both)
    torch.cuda.synchronize()
    # 48 additions to one float: their rounding is within the norm's tolerance
    assert float(one.abs().max()) > 0 and _close(both, one * (2 * times))


def test_more_threads_than_a_launch_holds():
    """2^30 rays and more (2^32 threads at four lanes a ray) go in several
    launches: rays with samples around the parts' ends, the others empty."""
    import torch
    print("[backward of 2^30 rays]", flush=True)
    if torch.cuda.mem_get_info()[0] < 90 << 30:
        pytest.skip("needs 90 GiB of device memory")
    o, d, g = _rays("tiny", 128)
    want = _grads(gpu_renderer("tiny"), o, d, g)
    n = (1 << 30) + 32
    big = [torch.zeros((n, 3), device="cuda") for _ in range(3)]
    for k, at in enumerate(((1 << 29) - 32, (1 << 30) - 32)):
        for whole, x in zip(big, (o, d, g)):
            whole[at:at + 64] = x[64 * k:64 * k + 64]
    got = _grads(gpu_renderer("tiny"), *big)
    torch.cuda.synchronize()
    assert all(float(b.abs().max()) > 0 and _close(a, b) for a, b in zip(got, want))


def test_capture_before_the_rows_are_there():
    """A captured backward whose workspace is at hand takes no memory for padded
    rows; replays with eager work between them, padded eager calls included."""
    import torch
    print("[padded rows: capture]", flush=True)
    n = 4096
    o, d, g = _rays("tiny", n)
    want = _grads(gpu_renderer("tiny"), o, d, g)
    r = gpu_renderer("tiny")
    r.set_deterministic(True)                             # takes the workspace, no rows
    _grads(r, o, d, g)
    r.set_deterministic(False)
    gt, gm = torch.zeros_like(want[0]), torch.zeros_like(want[1])
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        r.backward(o, d, g, gt, gm)
    for k in range(4):
        gt.zero_()
        gm.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert _close(gt, want[0]) and _close(gm, want[1])
        if k:
            eager = _grads(r, o, d, g)                    # padded: the rows are taken now
            assert _close(eager[0], want[0])
