"""Tiles of the three-kernel schedule: a layout takes 8x4x4, 8x8x4 or 8x8x8
nodes by the number of tiles its boxes make (at most 256).  Either side of both
limits, on ragged, walled and batched boxes, the state after three steps and
the exported fields are the bits of the fused schedule."""
import numpy as np
import pytest

import paper_2309_07801_amd as pkg
import workloads as WL

pytestmark = pytest.mark.gpu

# tiles of 8x4x4 and 8x8x4: (256, 128), (264, 132), (320, 160), (512, 256),
# (600, 300), ragged (72, 48), walls (90, 45), one node
LAYOUTS = [[(32, 32, 32, 0)], [(32, 33, 29, 0)], [(33, 31, 32, 0)], [(64, 32, 32, 0)],
           [(40, 40, 48, 0)], [(17, 23, 15, 0)], [(20, 12, 38, 3)], [(1, 1, 1, 0)],
           [(16, 24, 20, 0), (24, 9, 31, 2)], [(32, 32, 32, 0), (5, 7, 3, 0)]]


def _sim(shapes, storage):
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
    return pkg.Simulation(prm, rr, rb, u, seed=3, noise=1e-4, storage=storage)


@pytest.mark.parametrize("storage", [pkg.FP32, pkg.FP32_EXACT, pkg.FP16_SHIFT, pkg.BF16_CSHIFT])
@pytest.mark.parametrize("shapes", LAYOUTS)
def test_tiles_give_the_bits_of_the_fused_schedule(shapes, storage):
    got = []
    for schedule in (0, 1):
        sim = _sim(shapes, storage)
        sim.set_schedule(schedule)
        sim.step(3)
        state = sim.state_tensor().cpu().numpy().copy()
        got.append([state] + [v.cpu().numpy() for b in range(len(shapes))
                              for v in sim.moments(b).values()])
        sim.close()
    for a, b in zip(*got):
        assert np.array_equal(a, b)
