"""Handles with walls opened, stepped, re-tuned and closed one after another,
closed right after a step that may still be running, several alive at once:
each gives the bits of a handle that launches every kernel directly and waits
between its calls."""
import numpy as np
import pytest
import torch

import paper_2309_07801_amd as pkg
import workloads as WL

pytestmark = pytest.mark.gpu

SHAPES = [(40, 23, 30, 3), (33, 17, 24, 2), (70, 61, 37, 1), (24, 30, 90, 3), (64, 33, 20, 0)]


def _sim(shape):
    nx, ny, nz, walls = shape
    box = WL.two_phase_box((nx, ny, nz), 10.0, 1.0, 0.7, 0.01, 0.7, walls=walls)
    c = ((nx - 1) / 2.0, (ny - 1) / 2.0, (nz - 1) / 2.0)
    rr, rb, u = WL.droplet_fields(box, [c], [0.3 * min(nx, ny, nz)], u_carrier=(0.02, 0.0, 0.0))
    return pkg.Simulation([pkg.box_params_of(box)], [rr], [rb], [u], seed=3, noise=1e-5)


def _run(sim, k, wait):
    for change in (lambda: sim.set_schedule(2), lambda: sim.set_wall_mode(k % 4),
                   lambda: sim.set_compact_variant(k % 5), lambda: sim.set_schedule(1),
                   lambda: sim.set_schedule(0), lambda: sim.set_variant(k % pkg.num_variants())):
        sim.step(5)
        if wait:
            torch.cuda.synchronize()
        change()
    sim.step(4)


def test_handles_closed_while_their_steps_run():
    want = []
    for k, shape in enumerate(SHAPES):
        sim = _sim(shape)
        sim.set_graph(False)
        _run(sim, k, True)
        want.append(sim.checkpoint())
        torch.cuda.synchronize()
        sim.close()
    for turn in range(3):
        alive = []
        for k, shape in enumerate(SHAPES):
            sim = _sim(shape)
            _run(sim, k, False)
            got = sim.checkpoint()
            sim.step(6)  # pending when a later handle's turn closes this one
            alive.append(sim)
            if len(alive) > 2:
                alive.pop(0).close()
            assert torch.equal(got, want[k]), (turn, k)
        for sim in alive:
            sim.step(6)
            sim.close()
