"""The polled counts of agents per state and hazard class, at the edges of the
two ways they are taken: one block up to 16,384 agents, many beyond."""
import numpy as np
import pytest

from paper_1908_05232_amd import fps, inputs as I
from tests.gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("agents", [0, 1, 63, 1025, 4097, 16384, 16385])
def test_polled_counts_are_those_of_the_agents(agents):
    sc = I.shopping_centre(n=512, dx=0.25, seed=11, n_evac=agents, q_peak=60.0)
    sim = fps.Sim(sc)
    for steps in (0, 1, 150):
        sim.step(steps)
        d = sim.diag()
        assert d["n_agents"] == agents
        if not agents:
            assert sum(d["state_count"]) == 0 and sum(d["class_count"]) == 0
            continue
        A = sim.agents()
        inside = (A["state"] != 1) & (A["state"] != 7)
        assert list(d["state_count"]) == np.bincount(A["state"], minlength=8).tolist()
        assert list(d["class_count"]) == np.bincount(A["hr_class"][inside], minlength=6).tolist()
    say(f"{agents} agents: t {d['t']:.2f}, states {d['state_count']}, classes {d['class_count']}")
    assert d["step"] == 151 and d["t"] > 0.0
