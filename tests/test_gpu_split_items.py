"""How a pass deals out its items, beyond one workgroup per item.

Packs whose longest item outlasts the rest of a pass: the items are then shared out to two workgroups.  Parity with the
oracle where that split has its edges: a half without any key, a half of one key, one tile or an odd number of them per
head, groups of query heads (whose tiles follow one another in one item), head_dim below the tile width."""
import pytest

from test_gpu_parity import _full_check

pytestmark = pytest.mark.gpu

EDGES = [1, 63, 64, 65, 127, 128, 129, 191, 192, 193, 257]


@pytest.mark.parametrize("hq,hkv,d", [(2, 2, 128), (3, 1, 128), (2, 1, 104), (4, 2, 64), (2, 2, 40)])
@pytest.mark.parametrize("lengths", [EDGES, [449], [700, 64], [1100]])
def test_items_shared_by_two_workgroups(lengths, hq, hkv, d):
    _full_check(lengths, hq, hkv, d, seed=900 + d + len(lengths), magnitude_slack=True)


@pytest.mark.parametrize("hq,hkv,d", [(8, 8, 128), (16, 8, 104), (8, 8, 72)])
def test_many_short_items(hq, hkv, d):
    """More than a thousand short dK/dV items: the pass then draws them in persistent workgroups, several per workgroup."""
    lengths = [1 + (i * 37) % 131 for i in range(150)]
    _full_check(lengths, hq, hkv, d, seed=950 + d, magnitude_slack=True, slack_roundings=2)
