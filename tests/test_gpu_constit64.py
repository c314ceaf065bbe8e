"""The FP64 constitutive update at displacement gradients where the rotation
formulas of its eigen-decomposition have their special cases, against the
oracle: nothing to rotate, equal diagonal entries (a rotation by 45 degrees),
off-diagonal entries whose squares underflow, small and large strains.  The
update is a few hundred operations on entries of F (of order one) and the
return map shortens deviators without amplifying them: 1e-13 absolute."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _gradients(kind, d, n=64):
    rng = np.random.default_rng(5)
    a = rng.uniform(-1.0, 1.0, (n, d, d))
    eye = np.eye(d)
    if kind == "zero":
        return 0.0 * a
    if kind == "diagonal":
        return -0.01 * np.abs(a) * eye
    if kind == "equal":                 # equal diagonal, one or all off-diagonals
        g = -0.02 * eye + 1e-3 * a * (1.0 - eye)
        g[::2, 1:, :] *= eye[1:]
        return 0.5 * (g + g.transpose(0, 2, 1))
    if kind == "underflow":             # squares of the off-diagonals underflow
        return -0.01 * np.abs(a) * eye + 1e-170 * a * (1.0 - eye)
    if kind == "equal-underflow":
        return -0.02 * eye + 1e-170 * a * (1.0 - eye)
    scale = {"small": 1e-7, "large": 0.2}[kind]
    return scale * a - 0.3 * scale * eye


@pytest.mark.parametrize("d", [2, 3])
@pytest.mark.parametrize("kind", ["zero", "diagonal", "equal", "underflow", "equal-underflow", "small", "large"])
def test_constitutive_step_matches_oracle(kind, d):
    import torch

    import oracle
    import paper_2510_17335_amd as ddm
    print("case constitutive", kind, d, flush=True)
    sys.stdout.flush()
    g = _gradients(kind, d)
    n = len(g)
    cfg = ddm.make_config(d, 32, "f64", ppc=8.0, max_steps=4, checkpoint_every=2, sort_every=1)
    sim = ddm.Simulator(cfg, [ddm.make_instance(n, dt=1e-5, cohesion=0.0)])
    sim.init_state(np.random.default_rng(1).uniform(0.4, 0.6, (n, d)))
    state = sim.get_state()
    state[2 * d + d * d:, :n] = torch.from_numpy(g.reshape(n, d * d).T.copy()).to(state)
    sim.set_state(state)
    before = sim.packed_state(0)[:, 2 * d + d * d:].reshape(n, d, d)
    sim.step(1)
    assert sim.check().flags == 0
    after = sim.packed_state(0)[:, 2 * d + d * d:].reshape(n, d, d)
    want = np.stack([oracle.constitutive(f, 3.5e5, 0.3, 30.0)[1] for f in before])
    assert np.max(np.abs(after - want)) <= 1e-13
