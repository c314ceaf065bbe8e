"""The FP32 tile kernels at 1024 threads per workgroup (contexts of few tiles)
against the 256-thread kernels of the deterministic mode, at the particle
counts of one tile where the rounds change.  A second bed brings the context
to the size at which they are chosen."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

COUNTS = [1, 512, 513, 1023, 1024, 1025, 2049]
REST = 8192


def _sim(ddm, n, det, sort_every):
    cfg = ddm.make_config(3, 64, "f32", ppc=8.0, max_steps=4, checkpoint_every=2, sort_every=sort_every,
                          deterministic=det)
    return ddm.Simulator(cfg, [ddm.make_instance(n, dt=1e-5), ddm.make_instance(REST, dt=1e-5)])


def _positions(n):
    # one tile (cells 16 .. 19 per axis, base cell floor(64 x - 1/2)) and a bed of 10^3 cells
    rng = np.random.default_rng(n)
    x = np.concatenate([rng.uniform(16.51 / 64, 20.49 / 64, size=(n, 3)), rng.uniform(0.4, 0.55, size=(REST, 3))])
    return x.astype(np.float32).astype(np.float64)


@pytest.mark.parametrize("n", COUNTS)
def test_state_equals_narrow(n):
    """One FP32 sub-step: the same runs, FP64 window sums rounded to FP32; then
    two more, joined and one by one."""
    import torch

    import paper_2510_17335_amd as ddm
    print("case state", n, flush=True)
    sys.stdout.flush()
    states = []
    for det in (False, True):
        sim = _sim(ddm, n, det, 1)
        sim.init_state(_positions(n))
        sim.step(1)
        assert sim.check().flags == 0
        states.append(sim.get_state())
    assert torch.equal(states[0].view(torch.int32), states[1].view(torch.int32))
    packed = []
    for calls in ([3], [1, 1, 1]):
        sim = _sim(ddm, n, False, 4)
        sim.init_state(_positions(n))
        for k in calls:
            sim.step(k)
        assert sim.check().flags == 0
        packed.append((sim.packed_state(0), sim.packed_state(1)))
    for i in range(2):
        assert np.array_equal(packed[0][i], packed[1][i])


@pytest.mark.parametrize("n", COUNTS)
def test_gradient_equals_narrow(n):
    """FP32 gradients of a short rollout of a bed in shear and compression: the
    grid adjoint adds up to eight windows per node in another order (1e-7
    each), scaled by the conditioning of a short rollout, below 100 per step."""
    import torch

    import paper_2510_17335_amd as ddm
    print("case gradient", n, flush=True)
    sys.stdout.flush()
    target = np.full((2, 1600), 0.3)
    grads = []
    for det in (False, True):
        sim = _sim(ddm, n, det, 1)
        sim.init_state(_positions(n))
        state = sim.get_state().view(torch.float32)
        y = state[1:2].view(torch.int32).double()
        y = ((y + 2.0 ** 32) % 2.0 ** 32) * 2.0 ** -32
        state[3:6] = (y * torch.tensor([[2.0], [-1.0], [0.5]], dtype=y.dtype, device=y.device)).float()
        state[15:] = (1e-3 * torch.sin(40.0 * y * torch.arange(1, 10, device=y.device)[:, None])).float()
        state[19] -= 5e-3
        sim.set_state(state)
        sim.rollout(3)
        sim.loss(target)
        grads.append(sim.backward().cpu().numpy())
        assert sim.check().flags == 0
    g0, g1 = grads
    assert np.all(np.abs(g1).max(axis=1) > 0)
    assert np.all(np.abs(g0 - g1) <= 1e-4 * np.abs(g1).max(axis=1, keepdims=True)), (g0, g1)
