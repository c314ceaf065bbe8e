"""Workgroups of 512 and 1024 threads that take two and four tiles at once (where
a scattered bed occupies more tiles than are resident) against the 256-thread
kernels of the deterministic mode: tile counts at the switch (256 compute units
hold 256 or 512 such workgroups) and not divisible by two or four, a tile of
several rounds beside tiles of one particle, instances of different mass."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

N_GRID = 64


def _positions(rng, tiles, n, heavy):
    """n particles in exactly `tiles` tiles (4^3 cells each, base cell
    floor(64 x - 1/2)), `heavy` of them in one, every tile with one at least."""
    inner = np.stack(np.meshgrid(*[np.arange(2, 14)] * 3, indexing="ij"), -1).reshape(-1, 3)
    at = inner[rng.permutation(len(inner))[:tiles]]
    which = np.concatenate([np.arange(tiles), np.zeros(heavy, int), rng.integers(0, tiles, n - tiles - heavy)])
    x = (4 * at[which] + 0.51 + rng.uniform(0.0, 3.98, size=(n, 3))) / N_GRID
    return x.astype(np.float32).astype(np.float64)


# precision, then per instance (tiles, particles, particles of the heavy tile);
# from 4096 particles on FP32 takes 1024 threads
CASES = [
    ("f32", [(400, 700, 270), (112, 200, 0)]),
    ("f32", [(400, 700, 270), (113, 200, 0)]),
    ("f32", [(901, 2000, 600)]),
    ("f32", [(200, 3000, 1100), (57, 1400, 0)]),
    ("f32", [(700, 4096, 260), (301, 900, 300)]),
    ("f64", [(200, 900, 520), (56, 300, 0)]),
    ("f64", [(200, 900, 520), (59, 300, 0)]),
]


def _sim(ddm, prec, parts, det):
    cfg = ddm.make_config(3, N_GRID, prec, ppc=8.0, max_steps=4, checkpoint_every=2, sort_every=2, deterministic=det)
    inst = [ddm.make_instance(n, dt=1e-5, rho=1500.0 + 400.0 * i, E=3e5 * (1 + i)) for i, (_, n, _) in enumerate(parts)]
    sim = ddm.Simulator(cfg, inst)
    rng = np.random.default_rng(len(parts) + parts[0][0])
    sim.init_state(np.concatenate([_positions(rng, *p) for p in parts]))
    return sim


@pytest.mark.parametrize("prec,parts", CASES)
def test_state(prec, parts):
    """Two sub-steps (the second joined): the same runs, FP64 window sums
    rounded to FP32, so FP32 states agree bit for bit; FP64 ones to the order of
    sums of up to some hundred terms, 1e-16 each."""
    import torch

    import paper_2510_17335_amd as ddm
    print("case shared state", prec, parts, flush=True)
    sys.stdout.flush()
    states = []
    for det in (False, True):
        sim = _sim(ddm, prec, parts, det)
        sim.step(2)
        assert sim.check().flags == 0
        states.append(sim.get_state())
    if prec == "f32":
        assert torch.equal(states[0].view(torch.int32), states[1].view(torch.int32))
    else:
        for i in range(len(parts)):
            assert torch.linalg.norm(states[0] - states[1]) <= 1e-13 * torch.linalg.norm(states[1])


@pytest.mark.parametrize("prec,parts", CASES)
def test_gradient(prec, parts):
    """A short rollout of particles in shear and compression; the grid adjoint
    adds up to eight windows per node in another order (1e-7 and 1e-16 each),
    scaled by the conditioning of a short rollout, below 100 per step."""
    import torch

    import paper_2510_17335_amd as ddm
    print("case shared gradient", prec, parts, flush=True)
    sys.stdout.flush()
    target = np.full((len(parts), 1600), 0.3)
    grads = []
    for det in (False, True):
        sim = _sim(ddm, prec, parts, det)
        state = sim.get_state()
        y = torch.cat([sim.instance_state(state, i)[0] for i in range(len(parts))])[:, 1]
        cols = torch.cat([torch.arange(n, device=y.device) + off for (_, n, _), off in
                          zip(parts, np.cumsum([0] + [-(-n // 256) * 256 for _, n, _ in parts[:-1]]).tolist())])
        f = state if prec == "f64" else state.view(torch.float32)
        scale = torch.tensor([[2.0], [-1.0], [0.5]], dtype=y.dtype, device=y.device)
        wave = torch.arange(1, 10, device=y.device)[:, None]
        f[3:6, cols] = (y * scale).to(f.dtype)
        f[15:, cols] = (1e-3 * torch.sin(40.0 * y * wave)).to(f.dtype)
        f[19, cols] -= 5e-3
        sim.set_state(state)
        sim.rollout(3)
        sim.loss(target)
        grads.append(sim.backward().cpu().numpy())
        assert sim.check().flags == 0
    g0, g1 = grads
    assert np.all(np.abs(g1).max(axis=1) > 0)
    tol = 1e-8 if prec == "f64" else 1e-4
    assert np.all(np.abs(g0 - g1) <= tol * np.abs(g1).max(axis=1, keepdims=True)), (g0, g1)


@pytest.mark.parametrize("prec,parts", [CASES[2], CASES[4], CASES[6]])
def test_work_queue(prec, parts):
    """The same from persistent workgroups that draw groups of tiles from the
    queue (tile_workgroups), launched twice so that the queue's reset shows: FP32
    states bit for bit, FP64 to the order of sums."""
    import torch

    import paper_2510_17335_amd as ddm
    print("case shared queue", prec, parts, flush=True)
    sys.stdout.flush()
    states = []
    for workgroups in (0, 7, 97):
        cfg = ddm.make_config(3, N_GRID, prec, ppc=8.0, max_steps=8, checkpoint_every=2, sort_every=2)
        cfg.tile_workgroups = workgroups
        sim = ddm.Simulator(cfg, [ddm.make_instance(n, dt=1e-5, rho=1500.0 + 400.0 * i)
                                  for i, (_, n, _) in enumerate(parts)])
        rng = np.random.default_rng(5)
        sim.init_state(np.concatenate([_positions(rng, *p) for p in parts]))
        sim.step(5)
        assert sim.check().flags == 0
        states.append(sim.get_state())
    for other in states[1:]:
        if prec == "f32":
            assert torch.equal(states[0].view(torch.int32), other.view(torch.int32))
        else:
            assert torch.linalg.norm(states[0] - other) <= 1e-13 * torch.linalg.norm(states[0])
