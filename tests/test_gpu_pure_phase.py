"""Slabs (of the fused kernel) and tiles (of the interface kernel) whose phase
field is +1 or -1 throughout skip the interface stencils.  Pure and mixed
ones meet in every order along the march: layers one to five slabs thick, a
droplet smaller than a tile, no second phase at all, a perturbed bulk, with
and without walls.  The two kernels, which skip by different regions, give
the same bits in every exported field and state."""
import numpy as np
import pytest

import paper_2309_07801_amd as pkg
import workloads as WL

pytestmark = pytest.mark.gpu


def _fields(kind, box):
    z, y, x = np.meshgrid(np.arange(box.nz), np.arange(box.ny), np.arange(box.nx), indexing="ij")
    if kind == "layers":
        red = np.isin(z, (3, 9, 10, 17, 18, 19, 27, 28, 29, 30, 31))
    elif kind == "speck":
        red = (x - 20) ** 2 + (y - 11) ** 2 + (z - 18) ** 2 <= 4
    elif kind == "blue":
        red = np.zeros(box.shape, bool)
    else:  # a trace of blue in every red node of the upper half
        red = np.ones(box.shape, bool)
    rr = np.where(red, box.rho0_r, 0.0).astype(np.float32)
    rb = np.where(red, 0.0, box.rho0_b).astype(np.float32)
    if kind == "trace":
        rb = np.where(z > box.nz // 2, np.float32(1e-5), np.float32(0.0)).astype(np.float32)
    u = np.zeros((3,) + box.shape, np.float32)
    u[0], u[1] = 0.02, 0.01 * np.sin(2 * np.pi * x / box.nx)
    return rr, rb, u


@pytest.mark.parametrize("walls", [0, 3])
@pytest.mark.parametrize("kind", ["layers", "speck", "blue", "trace"])
def test_skipped_stencils_change_no_bit(kind, walls):
    box = WL.two_phase_box((43, 22, 38), 10.0, 1.0, 0.7, 0.02, 0.7, walls=walls)
    rr, rb, u = _fields(kind, box)
    got = []
    for schedule in (1, 0):
        sim = pkg.Simulation([pkg.box_params_of(box)], [rr], [rb], [u], seed=2, noise=1e-5)
        sim.set_schedule(schedule)
        out = []
        for n in (1, 3):
            sim.step(n)
            out.append(sim.state_tensor().cpu().numpy().copy())
            f = sim.moments(0)
            out += [f[k].cpu().numpy() for k in pkg.FIELDS]
        got.append(out)
        sim.close()
    for a, b in zip(*got):
        assert np.array_equal(a, b)


def test_field_export_serves_large_boxes_in_the_three_kernel_schedule():
    """From 2 Mi nodes on the three-kernel schedule takes its interface fields
    from the fused kernel's export: the same state as the fused schedule."""
    box = WL.two_phase_box((131, 127, 128), 10.0, 1.0, 0.7, 0.02, 0.7)
    assert box.nodes >= 2 << 20
    rr, rb, u = WL.droplet_fields(box, [(65.0, 63.0, 63.5)], [30.0], u_carrier=(0.02, 0.01, 0.0))
    got = []
    for schedule in (1, 0):
        sim = pkg.Simulation([pkg.box_params_of(box)], [rr], [rb], [u], seed=2, noise=1e-5)
        sim.set_schedule(schedule)
        sim.step(3)
        got.append(sim.state_tensor().cpu().numpy().copy())
        sim.close()
    assert np.array_equal(*got)
