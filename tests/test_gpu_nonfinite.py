"""Values that are not finite, or whose factors are not: a step that leaves NaN
discharges is a numeric fault at once, whatever shares the wave."""
import numpy as np
import pytest

from paper_1908_05232_amd import fps, inputs as I
from tests.gpu_util import say

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
