"""The pedestrian step with 16, 4 and 1 lanes an agent: the same bits.  The
number of lanes follows the agents of the launch, so a centre runs alone, and in
ensembles beside one whose crowd sets it."""
import numpy as np
import pytest

from paper_1908_05232_amd import fps, inputs as I
from tests.gpu_util import say

pytestmark = pytest.mark.gpu


# windows of obstacle cells: 81 (four words of mask), 25 (two), 9 (a cell a slot at most), 225 (no mask);
# agents: less than a group of four, ragged, a whole number of waves
@pytest.mark.parametrize("dx,agents", [(0.25, 3), (0.25, 1013), (0.5, 640), (2.0, 301), (0.15, 500)])
def test_lanes_do_not_change_the_bits(dx, agents):
    sc = I.shopping_centre(n=128, dx=dx, seed=17, n_evac=agents, q_peak=20.0)
    runs = []
    for crowd in (0, 21000, 270000):
        scs = [sc] + ([I.shopping_centre(n=768, dx=0.25, seed=18, n_evac=crowd)] if crowd else [])
        ens = fps.Ensemble(scs)
        ens.step(25)
        runs.append((ens[0].agents(), ens[0].diag()))
        ens.close()
    A, d = runs[0]
    moved = float(np.abs(A["x"] - sc.agents["x"]).max())
    say(f"dx {dx}, {agents} agents: t {d['t']:.3f}, moved up to {moved:.3f} m")
    assert moved > 0.0
    for B, e in runs[1:]:
        assert e["t"] == d["t"]
        for k in A:
            assert np.array_equal(A[k], B[k]), k
