"""Tile lists of a batch whose boxes' chunks differ in length, dealt to the
XCDs longest first: every box comes out as it does alone, with each launch
geometry of the compact schedule, one to nine boxes, with and without walls."""
import numpy as np
import pytest

import paper_2309_07801_amd as pkg
import workloads as WL

pytestmark = pytest.mark.gpu

SHAPES = [(70, 61, 37, 0), (24, 30, 90, 3), (33, 17, 64, 2), (9, 9, 9, 0), (128, 40, 24, 0),
          (17, 80, 11, 1), (3, 5, 130, 0), (64, 64, 64, 0), (40, 12, 70, 2)]


def _sim(shapes):
    prm, rr, rb, u = [], [], [], []
    for nx, ny, nz, walls in shapes:
        box = WL.two_phase_box((nx, ny, nz), 10.0, 1.0, 0.7, 0.01, 0.7, walls=walls)
        c = ((nx - 1) / 2.0, (ny - 1) / 2.0, (nz - 1) / 2.0)
        a, b, v = WL.droplet_fields(box, [c], [max(3.0, 0.3 * min(nx, ny, nz))],
                                    u_carrier=(0.02, 0.01 if not walls else 0.0, 0.0))
        prm.append(pkg.box_params_of(box))
        rr.append(a)
        rb.append(b)
        u.append(v)
    sim = pkg.Simulation(prm, rr, rb, u)
    sim.set_schedule(2)
    return sim


def _fields(sim, b):
    return [v.cpu().numpy() for v in sim.moments(b).values()]


@pytest.fixture(scope="module")
def alone():
    out = []
    for s in SHAPES:
        sim = _sim([s])
        sim.step(5)
        out.append(_fields(sim, 0))
        sim.close()
    return out


@pytest.mark.parametrize("variant", range(5))
@pytest.mark.parametrize("n", [1, 2, 3, 9])
def test_a_box_in_a_batch_is_the_box_alone(n, variant, alone):
    sim = _sim(SHAPES[:n])
    sim.set_variant((3 * variant + n) % pkg.num_variants())
    sim.set_compact_variant(variant)
    sim.step(5)
    for b in range(n):
        for got, want in zip(_fields(sim, b), alone[b]):
            assert np.array_equal(got, want), b
    sim.close()
