"""The two-level counting sort of the binning against the radix sort that the
deterministic mode uses: one FP32 sub-step from the same positions.  Both put a
cell's particles in id order there (the stable order of the first binning), the
run sums of the scatter follow that order, and their FP64 totals are rounded to
FP32, so the states agree bit for bit; an order that is not stable, a particle
in the wrong tile or a tile without its record changes them."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _positions(rng, n, dim, lo, hi):
    x = rng.uniform(lo, hi, size=(n, dim))
    return x.astype(np.float32).astype(np.float64)


# dim, grid, particles per instance, extent of the positions:
#   one workgroup and several of the tile table (4096 tiles each), ragged
#   instances of 1 and 257 particles, tiles around and beyond the 2048
#   particles that the per-tile kernel holds in LDS (one tile is 1/16 wide on a 64^3 grid)
CASES = [
    (2, 64, [2432], (0.1, 0.6)),
    (2, 16, [1, 300], (0.25, 0.7)),
    (3, 16, [128], (0.25, 0.7)),
    (3, 64, [5000, 1, 257], (0.2, 0.5)),
    (3, 128, [4099], (0.3, 0.6)),
    (3, 64, [2048], (0.2505, 0.3115)),
    (3, 64, [2049, 6000], (0.2505, 0.3115)),
]


@pytest.mark.parametrize("dim,n_grid,counts,extent", CASES)
def test_counting_sort_state_equals_radix_sort(dim, n_grid, counts, extent):
    import torch

    import paper_2510_17335_amd as ddm
    print("case", dim, n_grid, counts, extent, flush=True)
    sys.stdout.flush()
    rng = np.random.default_rng(7)
    x0 = np.concatenate([_positions(rng, n, dim, *extent) for n in counts])
    states = []
    for det in (False, True):
        cfg = ddm.make_config(dim, n_grid, "f32", ppc=8.0 if dim == 3 else 4.0, max_steps=4, checkpoint_every=2,
                              sort_every=1, deterministic=det)
        sim = ddm.Simulator(cfg, [ddm.make_instance(n, dt=1e-6) for n in counts])
        sim.init_state(x0)
        sim.step(1)
        assert sim.check().flags == 0
        states.append(sim.get_state())
        # the state is in key order (no particle moves a cell in 1e-6 s from rest)
        keys, perm = sim.bin_keys()
        assert np.all(np.diff(keys.astype(np.int64)) >= 0)
        assert np.array_equal(perm, np.arange(perm.size))
    assert torch.equal(states[0].view(torch.int32), states[1].view(torch.int32))
