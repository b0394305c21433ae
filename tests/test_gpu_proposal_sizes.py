"""The proposal's training step at batch sizes around its workgroups (64 rays,
16 a wave) and around the groups its partials are summed in (64), against the
bf16-operand oracle.

Tolerance: the oracle rounds the same operands to bfloat16 (relative error
2^-9 each); products and sums are float32 on one side and float64 on the
other, so a value near a rounding boundary can round apart, by 2^-8 of itself.
1e-2 in the norm covers such flips on a few of the operands."""
import numpy as np
import pytest

from helpers import to_gpu
from oracle import proposal as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 64, 65, 4097])
@pytest.mark.parametrize("phase", [1, 2])
def test_gradient_at_ragged_batches(n, phase):
    import torch
    from paper_2407_10482_amd.renderer import Proposal, Renderer
    print(f"[proposal batch {n} phase {phase}]", flush=True)
    rng = np.random.default_rng(n + phase)
    params = P.init_params(3)
    o = rng.uniform(-1, 1, size=(n, 3)).astype(np.float32)
    d = rng.normal(size=(n, 3)).astype(np.float32)
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    near = rng.uniform(0, 1, size=n)
    labels = np.stack([near, near + rng.uniform(0, 1, size=n), near + 0.1,
                       (rng.random(n) < 0.8).astype(np.float64)], 1).astype(np.float32)
    go, gd, gl, gp = to_gpu(o, d, labels, params)
    net = Proposal(gp, Renderer([16], 4))
    g, loss = net.grad(go, gd, gl, phase=phase, margin=0.05)
    f = P.forward(params, P.fourier(o, d), bf16_operands=True)
    valid = labels[:, 3] != 0
    ref_loss, g_out = P.loss_and_grad_out(f["out"], labels.astype(np.float64), valid, phase, 0.05)
    ref = P.backward(params, f, g_out, bf16_operands=True)
    got = g.cpu().numpy().astype(np.float64)
    assert abs(float(loss) - ref_loss) <= 1e-3 * max(1.0, abs(ref_loss))
    assert np.linalg.norm(got - ref) <= 1e-2 * np.linalg.norm(ref)
    # a training step with the same batch moves the weights by Adam's first step of that gradient
    before = gp.clone()
    net.train_step(go, gd, gl, 1e-3, phase=phase, margin=0.05)
    m1, v1 = (1.0 - np.float32(0.9)) * got, (1.0 - np.float32(0.99)) * got * got
    step = 1e-3 * (m1 / (1.0 - np.float32(0.9))) / (np.sqrt(v1 / (1.0 - np.float32(0.99))) + 1e-8)
    moved = (before - net.params).cpu().numpy().astype(np.float64)
    assert np.abs(moved - step).max() < 1e-6
    assert torch.allclose(net.m, 0.1 * g, rtol=1e-5, atol=1e-12)
