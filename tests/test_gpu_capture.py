"""A caller's own capture of fps_step: evacuee counts set after the capture are
those of the replay, and counts set right before a capture need nothing from the
host inside it."""
import numpy as np
import pytest
import torch

from paper_1908_05232_amd import fps
from tests.gpu_util import random_wet_dry, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", [1, 2])
@pytest.mark.parametrize("members", [1, 3])
def test_captured_steps_read_the_counts_of_the_replay(order, members):
    scs = [random_wet_dry(200 + 10 * k, 90, 0.5, seed=4 + k) for k in range(members)]
    for sc in scs:
        sc.desc.order = order
    counts = [[torch.full((90, 200 + 10 * k), n, dtype=torch.int32, device="cuda") for k in range(members)] for n in (7, 3)]
    torch.cuda.synchronize()
    runs = []
    for captured in (False, True):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            sim = fps.Sim(scs[0], stream=stream) if members == 1 else fps.Ensemble(scs, stream=stream)
            ms = [sim] if members == 1 else sim.members
            step = lambda: sim.step(2)
            step()
            stream.synchronize()
            if captured:
                graph = torch.cuda.CUDAGraph()
                with torch.cuda.graph(graph, stream=stream):
                    sim.step(2)
                step = graph.replay
            states = []
            for c in (None, counts[0], counts[1], None, counts[0]):
                for k, m in enumerate(ms):
                    m.set_occupancy(c[k] if c else None)
                step()
                stream.synchronize()
                states.append([f for m in ms for f in m.fields()[:3]])
        runs.append(states)
    eager, replayed = runs
    say(f"order {order}, {members} members: max|h| {np.abs(replayed[-1][0]).max():.4f}")
    for a, b in zip(eager, replayed):
        assert all(np.array_equal(x, y) for x, y in zip(a, b))


def test_counts_set_before_a_capture():
    sc = random_wet_dry(200, 90, 0.5, seed=4)
    some = torch.full((90, 200), 7, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    out = []
    for captured in (False, True):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            sim = fps.Sim(sc, stream=stream)
            sim.step(2)
            sim.set_occupancy(some)
            stream.synchronize()
            if captured:
                graph = torch.cuda.CUDAGraph()
                with torch.cuda.graph(graph, stream=stream):
                    sim.step(2)
                graph.replay()
            else:
                sim.step(2)
            stream.synchronize()
            out.append(sim.fields()[:3])
    assert all(np.array_equal(a, b) for a, b in zip(*out))
