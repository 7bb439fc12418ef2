"""Column tiles fitted to the box: every launch geometry of the fused kernel
and of the compact pull gives the same bits on boxes no nominal tile divides
(narrower than a tile, one node past one, whole rows, with and without
walls)."""
import numpy as np
import pytest

import paper_2309_07801_amd as pkg
import workloads as WL

pytestmark = pytest.mark.gpu

SHAPES = [(70, 61, 37, 0), (9, 130, 12, 0), (129, 33, 21, 0), (128, 7, 40, 0), (1, 40, 23, 0),
          (81, 67, 34, 3), (40, 23, 75, 2)]


def _sim(nx, ny, nz, walls, storage=pkg.FP32):
    box = WL.two_phase_box((nx, ny, nz), 10.0, 1.0, 0.7, 0.01, 0.7, walls=walls)
    c = ((nx - 1) / 2.0, (ny - 1) / 2.0, (nz - 1) / 2.0)
    rr, rb, u = WL.droplet_fields(box, [c], [max(3.0, 0.3 * min(nx, ny, nz))],
                                  u_carrier=(0.02, 0.01 if not walls else 0.0, 0.0))
    return pkg.Simulation([pkg.box_params_of(box)], [rr], [rb], [u], seed=3, noise=1e-4,
                          storage=storage)


def _state(sim):
    return sim.state_tensor().cpu().numpy().copy()


@pytest.mark.parametrize("nx,ny,nz,walls", SHAPES)
def test_every_geometry_gives_the_same_bits(nx, ny, nz, walls):
    steps = 3
    ref = _sim(nx, ny, nz, walls)
    ref.set_schedule(1)  # interface and collide kernels: no column tiles
    ref.step(steps)
    want = _state(ref)
    ref.close()
    compact = None
    for v in range(pkg.num_variants()):
        sim = _sim(nx, ny, nz, walls)
        sim.set_variant(v)
        sim.step(steps)
        assert np.array_equal(_state(sim), want), v
        sim.close()
        sim = _sim(nx, ny, nz, walls)
        sim.set_variant(v)
        sim.set_schedule(2)
        sim.set_compact_variant(v % 5, )
        sim.step(steps)
        got = _state(sim)
        sim.close()
        compact = got if compact is None else compact
        assert np.array_equal(got, compact), v


@pytest.mark.parametrize("storage", [pkg.FP32, pkg.FP32_EXACT, pkg.FP16_SHIFT, pkg.BF16_CSHIFT])
@pytest.mark.parametrize("nx", [1, 15, 16, 17, 49])
def test_padded_rows_of_the_compact_arrays(nx, storage):
    """Rows padded to 64 bytes where the buffers have the room (17 nodes: FP32
    and the mass-exact format, not the 16-bit ones; 1 node: none): one step
    per call of the compact schedule equals the population schedule."""
    out = []
    for schedule in (0, 2):
        sim = _sim(nx, 21, 18, 0, storage)
        sim.set_schedule(schedule)
        for _ in range(3):
            sim.step(1)
        out.append(_state(sim))
        sim.close()
    assert np.array_equal(*out)


@pytest.mark.parametrize("storage", [pkg.FP32, pkg.FP32_EXACT, pkg.FP16_SHIFT])
def test_d2q9_rows_of_whole_lines_and_ragged_ones(storage):
    """The D2Q9 step stores with the streaming hint where a row of stored words
    is whole cache lines and plainly elsewhere: a field that is uniform in x
    evolves alike, bit for bit, in boxes of 64 and of 77 columns."""
    out = []
    for nx in (64, 77):
        ny = 41
        box = WL.Box(nx=nx, ny=ny, nz=1, rho0_r=10.0, rho0_b=1.0, alpha_r=WL.alpha_heavy_2d(10.0),
                     alpha_b=WL.ALPHA_LIGHT_2D, nu_r=0.1, nu_b=0.1, sigma=0.01, beta=0.7)
        red = np.zeros(box.shape, bool)
        red[:, 9:24] = True
        u = np.zeros((3,) + box.shape, np.float32)
        u[0], u[1] = 0.03, 0.01 * np.sin(2 * np.pi * np.arange(ny) / ny)[None, :, None]
        sim = pkg.Simulation([pkg.box_params_of(box)], [np.where(red, 10.0, 0.0)],
                             [np.where(red, 0.0, 1.0)], [u], storage=storage, lattice="d2q9")
        sim.step(5)
        f = sim.moments(0, ("rho_r", "rho_b", "ux", "uy"))
        out.append({k: v.cpu().numpy()[0, :, :64] for k, v in f.items()})
        sim.close()
    for k in out[0]:
        assert np.array_equal(out[0][k], out[1][k]), k
