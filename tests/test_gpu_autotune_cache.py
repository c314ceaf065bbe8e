"""Contexts of one problem size whose sub-steps are other launches (the
deterministic mode, particle contact) share a cache file of ddm_autotune without
taking each other's line, nor one that names no options or other kernels."""
import sys

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _tuned(ddm, w, cache, **options):
    cfg, inst = ddm.from_workload(w, max_steps=8, checkpoint_every=4)
    for k, v in options.items():
        setattr(cfg, k, v)
    sim = ddm.Simulator(cfg, [inst])
    sim.init_state(W.bed_positions(w))
    return sim.autotune(cache), sim.launch()


def test_lines_are_not_shared(tmp_path):
    import paper_2510_17335_amd as ddm
    print("case autotune cache", flush=True)
    sys.stdout.flush()
    w = W.tiny(3, shovel=True)
    cache = str(tmp_path / "tune.txt")
    n = len(W.bed_positions(w))
    # what an earlier library wrote for this size: an interval that no probe gives
    old = f"ddmpm dim=3 n_grid={w.n_grid} prec=1 n_inst=1 particles={n} ppc={w.ppc} sort_every=64 tile_workgroups=0\n"
    open(cache, "w").write(old)
    options = ({"deterministic": 1}, {"particle_contact": 1}, {})
    got = [_tuned(ddm, w, cache, **o) for o in options]
    lines = open(cache).read().splitlines()
    assert len(lines) == 4 and lines[0] + "\n" == old
    for (r, launch), line in zip(got, lines[1:]):
        assert r in (2, 4, 8, 16, 32) and line.endswith(f" sort_every={r} tile_workgroups={launch[1]}")
    # a second look takes each its own line and adds none, whatever the file says beside it
    text = open(cache).read()
    for (r, _), line in zip(got, lines[1:]):
        text = text.replace(line, line.replace(f"sort_every={r} ", f"sort_every={3 + 2 * lines.index(line)} "))
    open(cache, "w").write(text)
    again = [_tuned(ddm, w, cache, **o)[0] for o in options]
    assert again == [5, 7, 9]
    assert len(open(cache).read().splitlines()) == 4
