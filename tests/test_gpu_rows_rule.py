"""The rows a wave marches before any tuning: what a member gets beside others must
leave it enough waves when the others have stopped."""
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
