"""The P2G adjoint in workgroups of one wave against the workgroups of four
waves of the deterministic mode, at the particle counts where the last wave of
an instance and its accumulator slots (64 waves) change."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [63, 64, 65, 193, 64 * 64, 64 * 64 + 1])
def test_gradient_equals_deterministic_mode(n):
    """FP64 gradients of a short rollout of a bed in shear and compression: they
    differ by the order of FP64 sums over some 10^4 terms of mixed sign (1e-12
    in all), scaled by the conditioning of a short rollout, below 100 per step."""
    import torch

    import paper_2510_17335_amd as ddm
    print("case waves", n, flush=True)
    sys.stdout.flush()
    x = np.random.default_rng(n).uniform(0.3, 0.5, size=(n + 65, 3))
    target = np.full((2, 1600), 0.3)
    grads = []
    for det in (False, True):
        cfg = ddm.make_config(3, 64, "f64", ppc=8.0, max_steps=4, checkpoint_every=2, sort_every=1, deterministic=det)
        sim = ddm.Simulator(cfg, [ddm.make_instance(n, dt=1e-5), ddm.make_instance(65, dt=1e-5)])
        sim.init_state(x)
        state = sim.get_state()
        state[3:6] = state[1:2] * torch.tensor([[2.0], [-1.0], [0.5]], dtype=state.dtype, device=state.device)
        state[15:] = 1e-3 * torch.sin(40.0 * state[:1] * torch.arange(1, 10, device=state.device)[:, None])
        state[19] -= 5e-3
        sim.set_state(state)
        sim.rollout(3)
        sim.loss(target)
        grads.append(sim.backward().cpu().numpy())
        assert sim.check().flags == 0
    g0, g1 = grads
    assert np.all(np.abs(g1).max(axis=1) > 0)
    assert np.all(np.abs(g0 - g1) <= 1e-8 * np.abs(g1).max(axis=1, keepdims=True)), (g0, g1)
