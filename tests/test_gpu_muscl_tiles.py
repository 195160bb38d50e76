"""The second-order march takes two rows a turn and strips of 60 columns: tiles of
odd and even heights, and sides at the edge of a strip, against the oracle and
against tiles of one row."""
import numpy as np
import pytest

from paper_1908_05232_amd import fps
from tests.gpu_util import random_wet_dry, say
from tests.test_gpu_flood import check_window

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ny", [1, 2, 3, 5, 7, 8, 9, 19, 63])
def test_row_counts_around_the_two_row_turn(ny):
    sc = random_wet_dry(130, ny, 0.5, seed=ny, bc=(0, 1, 0, 1))
    sc.desc.order = 2
    out = []
    for rows in (1, 2, 4, 8, 16, 64):
        sim = fps.Sim(sc)
        sim.set_rows_per_wave(rows)
        sim.step(4)
        out.append((sim.fields()[:3], sim.diag()))
    (ref, d0) = out[0]
    say(f"130 x {ny}: t {d0['t']:.4f}, outflow {d0['v_out']:.6g}")
    for f, d in out[1:]:
        assert all(np.array_equal(a, b) for a, b in zip(f, ref))
        assert d["t"] == d0["t"] and d["dt_next"] == d0["dt_next"]
        # FP64 sums in another order
        assert d["v_out"] == pytest.approx(d0["v_out"], rel=1e-10, abs=1e-12)


@pytest.mark.parametrize("nx", [59, 60, 61, 119, 120, 121])
def test_transmissive_east_side_at_the_edge_of_a_strip(oracle, nx):
    sc = random_wet_dry(nx, 21, 0.5, seed=nx, bc=(0, 1, 0, 0))
    sc.desc.order = 2
    sim = fps.Sim(sc)
    check_window(oracle, sim, sc, 100, f"order 2, random {nx}x21, open east", throughput=True)
    assert sim.diag()["v_out"] != 0.0
