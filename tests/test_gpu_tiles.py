"""The tile kernels at 512 threads per workgroup (small contexts) against the
256-thread kernels of the deterministic mode, at the particle counts of one
tile where the rounds and runs change: single particles, the edges of 256 and
512 slots, several rounds."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

COUNTS = [1, 255, 256, 257, 511, 512, 513, 1025]


def _sim(ddm, n, det, prec):
    cfg = ddm.make_config(3, 64, prec, ppc=8.0, max_steps=4, checkpoint_every=2, sort_every=1, deterministic=det)
    return ddm.Simulator(cfg, [ddm.make_instance(n, dt=1e-5), ddm.make_instance(3, dt=1e-5)])


def _positions(n):
    # one tile: cells 16 .. 19 per axis, base cell floor(64 x - 1/2)
    x = np.random.default_rng(n).uniform(16.51 / 64, 20.49 / 64, size=(n + 3, 3))
    return x.astype(np.float32).astype(np.float64)


@pytest.mark.parametrize("n", COUNTS)
def test_wide_tiles_state_equals_narrow(n):
    """One FP32 sub-step: the same runs, FP64 window sums rounded to FP32."""
    import torch

    import paper_2510_17335_amd as ddm
    print("case state", n, flush=True)
    sys.stdout.flush()
    states = []
    for det in (False, True):
        sim = _sim(ddm, n, det, "f32")
        sim.init_state(_positions(n))
        sim.step(1)
        assert sim.check().flags == 0
        states.append(sim.get_state())
    assert torch.equal(states[0].view(torch.int32), states[1].view(torch.int32))


@pytest.mark.parametrize("n", COUNTS)
def test_wide_tiles_gradient_equals_narrow(n):
    """FP64 gradients of a short rollout of a bed in shear and compression (in
    free fall from rest they would be zero): the two differ by the order of
    FP64 sums over at most a few thousand terms (1e-16 each, 1e-12 in all),
    scaled by the conditioning of a short rollout, below 100 per step."""
    import torch

    import paper_2510_17335_amd as ddm
    print("case gradient", n, flush=True)
    sys.stdout.flush()
    target = np.full((2, 1600), 0.3)
    grads = []
    for det in (False, True):
        sim = _sim(ddm, n, det, "f64")
        sim.init_state(_positions(n))
        state = sim.get_state()
        state[3:6] = state[1:2] * torch.tensor([[2.0], [-1.0], [0.5]], dtype=state.dtype, device=state.device)
        state[15:] = 1e-3 * torch.sin(40.0 * state[:1] * torch.arange(1, 10, device=state.device)[:, None])
        state[19] -= 5e-3
        sim.set_state(state)
        sim.rollout(3)
        loss = sim.loss(target)
        grads.append((loss.cpu().numpy(), sim.backward().cpu().numpy()))
    (l0, g0), (l1, g1) = grads
    assert np.allclose(l0, l1, rtol=1e-12, atol=0)
    assert np.all(np.abs(g0 - g1) <= 1e-8 * np.abs(g1).max(axis=1, keepdims=True)), (g0, g1)
