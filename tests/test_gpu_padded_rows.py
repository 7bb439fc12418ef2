"""Calls of many steps on the compact schedule's padded rows, where the compact
pull reads and writes them, against the FP64 oracle: widths that pad in every
storage (30, 33 and 49 nodes), in plain FP32 alone (17) and not at all (16),
periodic and between walls, one box and two unlike ones; and boxes under a body
force, whose pull has no short path, with wavefronts next to the interface and
away from it in one tile."""
import dataclasses

import numpy as np
import pytest

import paper_2309_07801_amd as pkg
import workloads as WL
from _common import FP32_BAR, bars_16bit, check, errors, gpu_fields, run_oracle, u_ref

pytestmark = pytest.mark.gpu

STORAGES = [pkg.FP32, pkg.FP32_PAIRS, pkg.FP32_EXACT, pkg.FP16_CSHIFT]


def _case(shape, walls=0, R=4.5, **kw):
    box = WL.two_phase_box(shape, 10.0, 1.0, 0.7, 0.01, 0.7, walls=walls)
    box = dataclasses.replace(box, **kw)
    c = tuple((n - 1) / 2.0 for n in shape)
    return box, WL.droplet_fields(box, [c], [R], u_carrier=(0.02, 0.0, 0.01 if not walls else 0.0))


def _sim(cases, storage):
    return pkg.Simulation([pkg.box_params_of(b) for b, _ in cases], [f[0] for _, f in cases],
                          [f[1] for _, f in cases], [f[2] for _, f in cases], seed=4, noise=1e-6,
                          storage=storage)


def _hold(cases, storage, calls):
    sim = _sim(cases, storage)
    sim.set_schedule(2)
    for n in calls:
        sim.step(n)
    bars = bars_16bit(storage) if storage == pkg.FP16_CSHIFT else (FP32_BAR,) * 3
    for k, (box, fl) in enumerate(cases):
        o = run_oracle(box, *fl, sum(calls), seed=4, noise=1e-6, box_index=k)[0]
        check(errors(gpu_fields(sim, k), o, box, u_ref(box, 0.02)), k, *bars)
    sim.close()


@pytest.mark.parametrize("storage", STORAGES)
@pytest.mark.parametrize("walls", [0, 3])
@pytest.mark.parametrize("nx", [16, 17, 30, 33, 49])
def test_many_steps_on_padded_rows_match_the_oracle(nx, walls, storage):
    _hold([_case((nx, 21, 18), walls)], storage, (3, 20, 7))


@pytest.mark.parametrize("storage", STORAGES)
def test_many_steps_on_padded_rows_of_a_batch(storage):
    _hold([_case((33, 21, 18), 1), _case((49, 17, 20), 0), _case((23, 16, 19), 2)], storage, (30,))


@pytest.mark.parametrize("storage", [pkg.FP32, pkg.FP32_PAIRS, pkg.FP32_EXACT])
@pytest.mark.parametrize("shape,walls", [((33, 21, 18), 3), ((49, 23, 17), 2), ((30, 19, 20), 1)])
def test_single_steps_on_padded_rows_between_walls_equal_the_population_schedule(shape, walls,
                                                                                 storage):
    out = []
    for schedule in (0, 2):
        sim = _sim([_case(shape, walls)], storage)
        sim.set_schedule(schedule)
        for _ in range(4):
            sim.step(1)
        out.append(sim.checkpoint().cpu().numpy())
        sim.close()
    assert np.array_equal(*out)


@pytest.mark.parametrize("storage", [pkg.FP32, pkg.FP32_EXACT])
@pytest.mark.parametrize("force", [dict(body_force=(2e-6, -1e-6, 1e-6)),
                                   dict(gravity=(0.0, 0.0, -2e-6), rho_ref=0.5)])
def test_forced_boxes_with_flat_and_curved_wavefronts_in_a_tile(force, storage):
    """A 70 x 40 column of tiles around a droplet of radius 7: most wavefronts
    hold no interface, some hold it whole, some in part."""
    _hold([_case((70, 40, 33), 0, 7.0, **force)], storage, (7, 33))
