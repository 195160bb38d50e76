"""The flood march's tile edges and the reduction of its partials: grids whose
partial count lies at the edges of the one-level and two-level reductions, row
counts around the four-row turn, and runs that need no evacuee counts."""
import numpy as np
import pytest
import torch

from paper_1908_05232_amd import fps
from tests.gpu_util import random_wet_dry, say

pytestmark = pytest.mark.gpu
BC = (1, 1, 1, 1)


def _run(sc, rows, steps, occ=None):
    sim = fps.Sim(sc)
    sim.set_rows_per_wave(rows)
    if occ is not None:
        sim.set_occupancy(occ)
    sim.step(steps)
    d, f = sim.diag(), sim.fields()
    sim.close()
    return d, f


# strips of 62 columns, one partial per strip and row band: 8192 partials are
# read in one level, more in chunks of 2048
@pytest.mark.parametrize("nx,ny", [(62 * 4, 2048), (62 * 4, 2049), (62 * 4 + 1, 1639), (62 * 5, 2048), (62 * 4, 2561)])
def test_partials_in_one_and_two_levels(nx, ny):
    sc = random_wet_dry(nx, ny, 0.5, seed=nx + ny, bc=BC, inflow=(2, 3, nx // 2))
    d1, f1 = _run(sc, 1, 3)
    d16, f16 = _run(sc, 16, 3)
    tiles = (nx + 61) // 62 * ny
    say(f"{nx} x {ny}: {tiles} partials, mass {d1['mass']:.9g}")
    for a, b in zip(f1, f16):
        assert np.array_equal(a, b)
    assert d1["dt_next"] == d16["dt_next"] and d1["t"] == d16["t"]
    # FP64 sums of FP32 depths in two orders: n eps of 64 bits, far below 1e-12
    exact = float(np.sum(f1[0].astype(np.float64))) * 0.25
    assert d1["mass"] == pytest.approx(exact, rel=1e-12)
    for k in ("v_out", "v_clip", "v_in"):
        assert d1[k] == pytest.approx(d16[k], rel=1e-10, abs=1e-12), k


@pytest.mark.parametrize("ny", [1, 2, 3, 4, 5, 7, 8, 9, 63, 66])
def test_row_counts_around_the_four_row_turn(ny):
    sc = random_wet_dry(130, ny, 0.5, seed=ny, bc=(0, 1, 0, 1))
    ref = _run(sc, 1, 4)
    for rows in (2, 4, 8, 16, 64):
        d, f = _run(sc, rows, 4)
        assert all(np.array_equal(a, b) for a, b in zip(f, ref[1])), (ny, rows)
        assert d["dt_next"] == ref[0]["dt_next"]


def test_no_counts_equals_zero_counts():
    sc = random_wet_dry(200, 90, 0.5, seed=4)
    zero = torch.zeros(90, 200, dtype=torch.int32, device="cuda")
    some = zero.clone()
    some[::3, ::2] = 7
    plain = _run(sc, 4, 6)[1]
    assert all(np.array_equal(a, b) for a, b in zip(plain, _run(sc, 4, 6, zero)[1]))
    rough = _run(sc, 4, 6, some)[1]
    assert not np.array_equal(plain[1], rough[1])
    # counts set, then cleared, between steps
    sim = fps.Sim(sc)
    sim.step(2)
    sim.set_occupancy(some)
    sim.set_occupancy(None)
    sim.step(4)
    assert all(np.array_equal(a, b) for a, b in zip(plain, sim.fields()))


# 64 blocks of 256 cells count themselves in the copy back, 65 leave it to a launch
@pytest.mark.parametrize("nx,ny", [(16, 16), (128, 128), (129, 128), (300, 200)])
def test_odd_calls_return_the_state_to_the_callers_buffers(nx, ny):
    """Calls of one and three steps (the state ends in the scratch buffers)
    against one call, alone and beside a member that stopped on an odd step."""
    scs = [random_wet_dry(nx, ny, 0.5, seed=nx + k, bc=BC, inflow=(2, 3, nx // 2)) for k in (0, 1)]
    whole = _run(scs[0], 1, 12)[1]
    ens = fps.Ensemble(scs)
    ens.step(1)
    ens[1].set_end_time(ens[1].diag()["t"] * 1.5)      # stops in the next step
    for n in (1, 3, 1, 5, 1):
        ens.step(n)
        if n == 3:
            stopped = ens[1].fields()
    say(f"{nx} x {ny}: member 1 stopped at step {ens[1].diag()['step']}")
    assert ens[1].diag()["active"] == 0 and ens[0].diag()["step"] == 12
    for a, b in zip(ens[0].fields(), whole):
        assert np.array_equal(a, b)
    for a, b in zip(ens[1].fields(), stopped):
        assert np.array_equal(a, b)
