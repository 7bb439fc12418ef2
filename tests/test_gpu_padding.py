"""The stored state's bytes are functions of its nodes: the padding between
boxes and at the planes' ends is zero whatever ran before -- the compact
schedule's arrays, of other rows and planes, lie in the second population
buffer, which the next step of another schedule makes the state."""
import numpy as np
import pytest
import torch

import paper_2309_07801_amd as pkg
import workloads as WL

pytestmark = pytest.mark.gpu

SHAPES = [(150, 61, 37, 0), (133, 50, 21, 3)]


def _sim(storage):
    prm, rr, rb, u = [], [], [], []
    for nx, ny, nz, walls in SHAPES:
        box = WL.two_phase_box((nx, ny, nz), 10.0, 1.0, 0.7, 0.01, 0.7, walls=walls)
        c = ((nx - 1) / 2.0, (ny - 1) / 2.0, (nz - 1) / 2.0)
        a, b, v = WL.droplet_fields(box, [c], [7.0], u_carrier=(0.02, 0.0, 0.0))
        prm.append(pkg.box_params_of(box))
        rr.append(a)
        rb.append(b)
        u.append(v)
    return pkg.Simulation(prm, rr, rb, u, seed=3, noise=1e-5, storage=storage)


def _state(sim):
    return sim.state_tensor().cpu().numpy().copy()


@pytest.mark.parametrize("schedule", [0, 1])
@pytest.mark.parametrize("storage", [pkg.FP32, pkg.FP16_SHIFT, pkg.BF16_SHIFT, pkg.FP32_EXACT,
                                     pkg.FP32_PAIRS, pkg.FP16_CSHIFT, pkg.BF16_CSHIFT])
def test_padding_of_the_state_is_zero_after_any_history(storage, schedule):
    plain = _sim(storage)
    plain.set_schedule(schedule)
    plain.step(5)
    want = _state(plain)
    plain.close()
    sim = _sim(storage)
    sim.autotune(reps=1)  # runs the compact schedule's kernels on the other buffer
    sim.set_schedule(schedule)
    sim.step(5)
    assert np.array_equal(_state(sim), want)
    sim.set_schedule(2)
    sim.step(4)
    populations = _state(sim)
    sim.set_schedule(schedule)
    sim.step(3)  # a captured pair and a direct step
    got = _state(sim)
    # from the same populations, with no compact state before
    fresh = _sim(storage)
    fresh.set_schedule(schedule)
    fresh.load_state(torch.from_numpy(populations).to(fresh.device))
    fresh.step(3)
    assert np.array_equal(got, _state(fresh))
    sim.close()
    fresh.close()
