"""Values that are not finite, or whose factors are not: a step that leaves NaN
discharges is a numeric fault at once, whatever shares the wave; a film of still
water has no friction however thin it is; a bed of infinite height is a wall."""
import numpy as np
import pytest
import torch

from paper_1908_05232_amd import fps, inputs as I
from tests.gpu_util import random_wet_dry, say

pytestmark = pytest.mark.gpu


# 40 x 4: one wave; 248 x 2049 at a row a wave: 8,196 partials, reduced in two levels
@pytest.mark.parametrize("nx,ny,calm", [(40, 4, False), (40, 4, True), (248, 2049, True)])
@pytest.mark.parametrize("order", [1, 2])
def test_overflowed_speeds_are_a_fault_in_the_step_that_made_them(nx, ny, calm, order):
    """u * u + v * v overflows in a pool ten columns wide: the friction makes its
    discharges NaN, its depths stay finite.  With a calm pool in the same wave, or
    with nothing else wet anywhere."""
    h, hu, z = np.zeros((ny, nx)), np.zeros((ny, nx)), np.full((ny, nx), 2.0)
    h[:4, :10], hu[:4, :10], z[:4, :10] = 1.0, 1.5e19, 0.0
    if calm:
        h[:, 30:], z[:, 30:] = 0.5, 0.0
    sc = I.Scenario(desc=I.GridDesc(nx=nx, ny=ny, dx=0.5, dy=0.5, bc=(1, 1, 1, 1), order=order), h=h, qx=hu,
                    qy=hu.copy(), z=z)
    sim = fps.Sim(sc)
    sim.set_rows_per_wave(4 if ny == 4 else 1)
    sim.step(1)
    d, (h1, qx1, _, _) = sim.diag(check=False), sim.fields()
    say(f"{nx} x {ny}, order {order}: status {d['status']}, {int(np.isnan(qx1).sum())} NaN discharges, "
        f"{int(np.isnan(h1).sum())} NaN depths")
    assert np.isnan(qx1).any() and np.isfinite(h1).all()
    assert d["rc"] == fps.FPS_E_NUMERIC


# dt g n^2 h^(-4/3) is 1.9e23, 7.5e20 and 9.8e20: over a speed held at 1e-18 it overflows
@pytest.mark.parametrize("h_dry,depth,dt_max,dx,people", [
    (1e-20, 1e-19, 1.0, 0.5, 0), (1e-13, 2e-13, 1e6, 100.0, 0), (1e-16, 5e-16, 1.0, 0.5, 20)])
@pytest.mark.parametrize("order", [1, 2])
def test_film_of_still_water_stays_still(h_dry, depth, dt_max, dx, people, order):
    nx, ny = 70, 9
    zero = np.zeros((ny, nx))
    d = I.GridDesc(nx=nx, ny=ny, dx=dx, dy=dx, h_dry=h_dry, dt_max=dt_max, n_base=0.03, order=order)
    sim = fps.Sim(I.Scenario(desc=d, h=zero + depth, qx=zero, qy=zero, z=zero))
    if people:
        sim.set_occupancy(torch.full((ny, nx), people, dtype=torch.int32, device="cuda"))
    sim.step(3)
    h, qx, qy, _ = sim.fields()
    say(f"film of {depth} m: max|q| {np.abs(qx).max()}, {np.abs(qy).max()}, t {sim.diag()['t']}")
    assert np.all(h == np.float32(depth)) and np.all(qx == 0) and np.all(qy == 0)


@pytest.mark.parametrize("order,depth", [(1, 0.0), (2, 0.0), (1, 0.01)])
def test_infinite_bed_is_a_wall(order, depth):
    """Blocks of cells whose bed is +inf, alone, in pairs, in large blocks and along the
    sides, against the same cells 1,000 km high: the same bits everywhere else, and the
    water that lies on them stays."""
    nx, ny = 130, 70
    sc = random_wet_dry(nx, ny, 0.5, seed=8, bc=(0, 1, 0, 1))
    sc.desc.order = order
    block = I.rng_of(9).random((ny, nx)) < 0.05
    for j, i in ((10, 20), (30, 55), (40, 0), (0, 80), (64, 118)):
        block[j:j + 6, i:i + 12] = True
    for f in (sc.h, sc.qx, sc.qy):
        f[block] = 0.0
    out = []
    for height, held in ((1e6, 0.0), (np.inf, depth)):
        sc.z[block] = height
        sc.h[block] = held
        sim = fps.Sim(sc)
        sim.step(20)
        out.append((sim.fields()[:3], sim.diag()["t"]))
    (ref, t), (got, ti) = out
    say(f"order {order}, {int(block.sum())} cells, t {t:.4f} and {ti:.4f}")
    assert t == ti
    for a, b in zip(ref, got):
        assert np.array_equal(a[~block], b[~block])
    assert np.all(got[0][block] == np.float32(depth)) and np.all(got[1][block] == 0) and np.all(got[2][block] == 0)
