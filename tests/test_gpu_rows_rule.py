"""The rows a wave marches before any tuning: what a member gets beside others must
leave it enough waves when the others have stopped, and the lines of the rule lie
between sizes measured on either side, so that sizes nearby get the same."""
import numpy as np
import pytest

from paper_1908_05232_amd import fps, inputs as I
from tests.gpu_util import say

pytestmark = pytest.mark.gpu


def rows_of(sizes):
    scs = [I.lake_at_rest(n, n, 0.5, seed=3) for n in sizes]
    ens = fps.Ensemble(scs)
    rows = [m.rows_per_wave() for m in ens.members]
    ens.close()
    return rows


# grids a side; strips are 62 columns wide
@pytest.mark.parametrize("sizes", [[256] * 32, [512] * 16, [1024, 512, 256, 716] * 4, [700] * 24, [128] * 36, [1024] * 12])
def test_an_average_member_left_alone_keeps_512_waves(sizes):
    rows = rows_of(sizes)
    waves = [-(-n // 62) * -(-n // h) for n, h in zip(sizes, rows)]
    say(f"{len(sizes)} members: rows {sorted(set(rows))}, {sum(waves)} waves, {sum(waves) / len(sizes):.0f} a member")
    assert len(set(rows)) == 1
    assert max(rows) <= 4 or sum(waves) >= 512 * len(sizes)


@pytest.mark.parametrize("n,rows", [(400, 1), (440, 2), (480, 2), (510, 2), (512, 2), (620, 2), (768, 2), (860, 4),
                                    (1024, 4), (1400, 4), (1600, 8), (2048, 8), (2400, 16), (3000, 16)])
def test_rows_of_one_grid(n, rows):
    sim = fps.Sim(I.Scenario(desc=I.GridDesc(nx=n, ny=n, dx=0.5, dy=0.5), h=np.zeros((n, n)), qx=np.zeros((n, n)),
                             qy=np.zeros((n, n)), z=np.zeros((n, n))))
    assert sim.rows_per_wave() == rows
    sim.close()
