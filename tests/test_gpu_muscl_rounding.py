"""Rounding of the second-order update on long waves, where nothing but rounding is
left between it and the FP64 oracle: the root mean square of the difference after
eight steps, averaged over seeds.  The bed-slope term takes the surface's change
across a cell from the rounded values that the faces took; from the unrounded slope
it did not match them, and the difference added up from step to step."""
import numpy as np
import pytest

from paper_1908_05232_amd import fps, inputs as I
from tests.gpu_util import say

pytestmark = pytest.mark.gpu
N, STEPS, SEEDS = 384, 8, 6


def waves(seed, flux):
    rng = I.rng_of(seed)
    y, x = np.mgrid[0:N, 0:N] / N

    def wave(amp):
        return amp / 3 * sum(np.cos(6.28 * a) * np.sin(6.28 * ((1 + 9 * b) * x + (1 + 9 * c) * y + d))
                             for a, b, c, d in rng.random((6, 4)))

    z = wave(0.1)
    h = np.maximum(0.25 + wave(0.2) - z, 0.0)
    q = [h * wave(0.6) * (h > 0.01) for _ in range(2)]
    f32 = [a.astype(np.float32).astype(np.float64) for a in (h, *q, z)]
    desc = I.GridDesc(nx=N, ny=N, dx=0.25, dy=0.25, order=2, flux=flux)
    return I.Scenario(desc=desc, h=f32[0], qx=f32[1], qy=f32[2], z=f32[3])


def rounding(oracle, flux):
    """Mean square of the difference in h and in the discharges, over the seeds."""
    eh = eq = 0.0
    for seed in range(SEEDS):
        sc = waves(seed, flux)
        sim, ref = fps.Sim(sc), oracle.OracleSim(sc)
        for _ in range(STEPS):
            sim.step(1)
            ref.fv_step(sim.diag()["dt_last"])
        (h, qx, qy, _), (hr, qxr, qyr, _) = sim.fields(), ref.fields()
        eh += np.mean((h - hr) ** 2) / SEEDS
        eq += np.mean(((qx - qxr) ** 2 + (qy - qyr) ** 2) / 2) / SEEDS
        sim.close()
    return float(np.sqrt(eh)), float(np.sqrt(eq))


# the bars: the scheme with general faces and the bed slope in squares has 1.569e-8 m and
# 1.707e-8 m^2/s with HLLC, 1.620e-8 and 1.747e-8 with HLL; the unrounded slope 1.583e-8 and 1.796e-8 with HLLC
@pytest.mark.parametrize("flux,bar_h,bar_q", [(0, 1.575e-8, 1.715e-8), (1, 1.625e-8, 1.755e-8)])
def test_rounding_is_no_more_than_that_of_the_plain_form(oracle, flux, bar_h, bar_q):
    eh, eq = rounding(oracle, flux)
    say(f"flux {flux}: rms of h {eh:.4e} m, of the discharges {eq:.4e} m^2/s")
    assert eh <= bar_h and eq <= bar_q
