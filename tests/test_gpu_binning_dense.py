"""Tiles of more particles than the per-tile ordering of the binning holds in LDS
(2048): the order against the radix sort of the deterministic mode, and that the
time grows with the particle count and not with its square."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _sim(ddm, counts, x, det, prec="f32", dim=3):
    cfg = ddm.make_config(dim, 64, prec, ppc=8.0 if dim == 3 else 4.0, max_steps=4, checkpoint_every=2, sort_every=1,
                          deterministic=det)
    sim = ddm.Simulator(cfg, [ddm.make_instance(n, dt=1e-6) for n in counts])
    sim.init_state(x)
    return sim


def _tile_positions(rng, n, dim, cells):
    # the first `cells` cells per axis of the tile of cells 16 .. 19 (base cell floor(64 x - 1/2)), in no order
    x = rng.uniform(16.51 / 64, (16.49 + cells) / 64, size=(n, dim))
    return x.astype(np.float32).astype(np.float64)


# dimension, particles of each instance, cells per axis that they fill: sorting
# steps of 1024, numbers of slot digits (up to 256^2 slots and beyond), one cell
@pytest.mark.parametrize("dim,counts,cells", [
    (3, [3072, 3073], 4),
    (3, [20000, 5], 4),
    (3, [5, 70000], 4),
    (3, [9000], 1),
    (2, [2500, 4097], 4),
])
def test_order_equals_radix_sort(dim, counts, cells):
    """One FP32 sub-step: the order of a cell's particles decides its FP32 sums,
    so the states agree bit for bit."""
    import torch

    import paper_2510_17335_amd as ddm
    print("case dense order", dim, counts, cells, flush=True)
    sys.stdout.flush()
    rng = np.random.default_rng(11)
    x = np.concatenate([_tile_positions(rng, n, dim, cells) for n in counts])
    states = []
    for det in (False, True):
        sim = _sim(ddm, counts, x, det, dim=dim)
        sim.step(1)
        assert sim.check().flags == 0
        states.append(sim.get_state())
        keys, perm = sim.bin_keys()
        assert np.all(np.diff(keys.astype(np.int64)) >= 0)
        assert np.array_equal(perm, np.arange(perm.size))
    assert torch.equal(states[0].view(torch.int32), states[1].view(torch.int32))


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_time_is_linear(prec):
    """Ten times the particles of a tile take ten times the steps (and one
    more pass over them where the slot numbers get another digit, 4 / 3); a
    comparison with all others would take a hundred times the time."""
    import paper_2510_17335_amd as ddm
    rng = np.random.default_rng(12)
    ms = []
    for n in (20000, 200000):
        print("case dense time", prec, n, flush=True)
        sys.stdout.flush()
        sim = _sim(ddm, [n], _tile_positions(rng, n, 3, 4), False, prec)
        sim.step(1)
        sim.set_timing(groups=["binning"])
        sim.step(2)
        total, count = sim.read_timing()["binning"]
        assert sim.check().flags == 0
        ms.append(total / count)
    print("ms per binning", ms, flush=True)
    assert ms[1] <= 30.0 * ms[0]


@pytest.mark.parametrize("dim,n_grid", [(2, 64), (3, 64)])
@pytest.mark.parametrize("tiles", [1, 2, 8, 9, 64])
def test_waves_of_several_tiles(dim, n_grid, tiles):
    """Waves whose 64 lanes lie in a given number of tiles, by turns: the first
    eight are counted tile by tile, the lanes of further ones each by itself.
    The state is that of the radix sort, bit for bit."""
    import torch

    import paper_2510_17335_amd as ddm
    print("case waves", dim, tiles, flush=True)
    sys.stdout.flush()
    rng = np.random.default_rng(tiles)
    inner = np.stack(np.meshgrid(*[np.arange(3, 12)] * dim, indexing="ij"), -1).reshape(-1, dim)
    n = 700
    at = inner[rng.permutation(len(inner))[:64]]
    lane = np.arange(n) % 64 % tiles + (np.arange(n) // 64 * tiles) % 64
    x = (4 * at[lane % 64] + 0.51 + rng.uniform(0.0, 3.98, size=(n, dim))) / n_grid
    x = x.astype(np.float32).astype(np.float64)
    states = []
    for det in (False, True):
        sim = _sim(ddm, [n], x, det, dim=dim)
        sim.step(1)
        assert sim.check().flags == 0
        states.append(sim.get_state())
    assert torch.equal(states[0].view(torch.int32), states[1].view(torch.int32))
