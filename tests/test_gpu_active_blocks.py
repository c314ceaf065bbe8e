"""The blocks around occupied tiles (those that can receive mass) at the edges
of the grid, of a row of tiles and of the 4096 tiles that one workgroup of the
tile table holds: scattered particles, one FP32 sub-step, against the radix sort
of the deterministic mode, which marks them tile by tile.  A block left out
loses its mass.  Bit for bit, as the arithmetic of both is the same."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,n_grid,counts,extent", [
    (2, 16, [9, 40], (0.2, 0.8)),
    (2, 256, [1500], (0.03, 0.97)),
    (3, 16, [12, 200], (0.2, 0.8)),
    (3, 64, [700, 90], (0.07, 0.93)),
    (3, 128, [1500], (0.04, 0.96)),
])
def test_state_equals_deterministic_mode(dim, n_grid, counts, extent):
    import torch

    import paper_2510_17335_amd as ddm
    print("case", dim, n_grid, counts, flush=True)
    sys.stdout.flush()
    rng = np.random.default_rng(3)
    x0 = np.concatenate([rng.uniform(*extent, size=(n, dim)) for n in counts]).astype(np.float32).astype(np.float64)
    states = []
    for det in (False, True):
        cfg = ddm.make_config(dim, n_grid, "f32", ppc=8.0 if dim == 3 else 4.0, max_steps=4, checkpoint_every=2,
                              sort_every=1, deterministic=det)
        sim = ddm.Simulator(cfg, [ddm.make_instance(n, dt=1e-6) for n in counts])
        sim.init_state(x0)
        sim.step(1)
        assert sim.check().flags == 0
        states.append(sim.get_state())
    assert torch.equal(states[0].view(torch.int32), states[1].view(torch.int32))
