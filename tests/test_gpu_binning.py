"""The neighbour bins after a step against the oracle's stable counting sort, at
the edges of the paths: one to sixteen tiles of the LDS binning, its largest
numbers of bins and agents, and the grids just past them, which are scanned by
many blocks."""
import numpy as np
import pytest

from paper_1908_05232_amd import fps, inputs as I
from tests.gpu_util import say

pytestmark = pytest.mark.gpu


# cells a side, bins (4 x 4 cells each), agents
@pytest.mark.parametrize("n,nbins,agents", [
    (512, 128 ** 2, 2000), (516, 129 ** 2, 2000), (724, 181 ** 2, 8192), (728, 182 ** 2, 1), (1024, 256 ** 2, 8192),
    (724, 181 ** 2, 8193), (1028, 257 ** 2, 500), (2048, 512 ** 2, 3000), (2052, 513 ** 2, 300)])
def test_bins_at_the_edges_of_the_paths(oracle, n, nbins, agents):
    sc = I.shopping_centre(n=n, dx=0.25, seed=n, n_evac=agents, q_peak=20.0)
    sim = fps.Sim(sc)
    P = oracle.make_params(sc.desc, sc.ped)
    for _ in range(3):
        sim.step(2)
        A = sim.agents()
        bs, perm = sim.bins()
        bs_ref, perm_ref = oracle.build_bins(P, A["x"], A["y"], A["state"])
        assert len(bs) == nbins + 1
        assert np.array_equal(bs, bs_ref) and np.array_equal(perm, perm_ref)
    say(f"{n}^2, {agents} agents: {len(perm)} in {nbins} bins")


def test_crowded_bins_keep_the_stable_order(oracle):
    """3,000 agents on a few cells: hundreds to a bin."""
    sc = I.shopping_centre(n=640, dx=0.25, seed=3, n_evac=3000)
    A = sc.agents
    for k in ("x", "y"):
        v = A[k]
        v[:] = v[:1] + (v - v[:1]) * np.float32(0.01)
    sim = fps.Sim(sc)
    P = oracle.make_params(sc.desc, sc.ped)
    sim.step(3)
    A = sim.agents()
    bs, perm = sim.bins()
    bs_ref, perm_ref = oracle.build_bins(P, A["x"], A["y"], A["state"])
    say(f"most in a bin: {int(np.diff(bs).max())}")
    assert np.diff(bs).max() > 100
    assert np.array_equal(bs, bs_ref) and np.array_equal(perm, perm_ref)


def test_stopped_member_with_many_bins_keeps_them(oracle):
    """A member beyond the LDS binning (8,300 agents; 66,049 bins in 17 chunks) stops
    while one with as many bins, and one binned in LDS, step on."""
    scs = [I.shopping_centre(n=n, dx=0.25, seed=n + k, n_evac=m, q_peak=20.0)
           for k, (n, m) in enumerate(((1028, 8300), (64, 50), (1028, 9000)))]
    ens = fps.Ensemble(scs)
    ens[0].set_end_time(1.0)
    ens.step(60)
    assert ens[0].diag()["active"] == 0 and ens.active() == 2
    for step in (0, 7):
        ens.step(step)
        for k, sc in enumerate(scs):
            P, A = oracle.make_params(sc.desc, sc.ped), ens[k].agents()
            bs, perm = ens[k].bins()
            bs_ref, perm_ref = oracle.build_bins(P, A["x"], A["y"], A["state"])
            assert np.array_equal(bs, bs_ref) and np.array_equal(perm, perm_ref)
    say(f"stopped at t = {ens[0].diag()['t']:.3f}")
