"""The end of a queue: where the chains of a list are alike, the last round and a half of items goes by cost, not chain by chain."""
import numpy as np
import pytest

import paper_2504_20490_amd as A


def _steps(kind, items):
    length, tile = items[:, 1].astype(np.int64), items[:, 2].astype(np.int64)
    steps = -(-(length - tile * 128) // 64) if kind == A.LIST_DKV else -(-np.minimum(length, (tile + 1) * 128) // 64)
    return np.where(tile < 0, 0, steps)


@pytest.mark.parametrize("kind,resident", [(A.LIST_FWD, 64), (A.LIST_DQ, 64), (A.LIST_DKV, 32)])
@pytest.mark.parametrize("lengths,heads,rows,keys", [
    ([2697] * 5, 8, True, True),            # 110 items a queue
    ([832] * 13, 8, True, True),            # thirteen steps: the least that counts in the rows lists
    ([768] * 13, 8, False, True),           # twelve
    ([640] * 20, 8, False, True),           # ten: the least in the dK/dV list
    ([576] * 20, 8, False, False),
    ([2048] * 10, 8, True, True),           # five rounds of the dK/dV list
    ([2048] * 11, 8, True, False),
    ([2048] * 21, 8, False, False),         # more than five of the others
    ([2048, 200] * 4, 8, False, False),     # the last chains are cheap anyway
    ([1500] * 4, 8, False, True)])          # 48 items a queue: no more than the other passes run at once
def test_last_items_of_a_queue(kind, resident, lengths, heads, rows, keys):
    by_cost = keys if kind == A.LIST_DKV else rows
    cu, _, _ = A.build_cu_seqlens(lengths)
    items = A.schedule(kind, cu, heads, heads)
    want = {(int(cu[s]), n, t, h) for s, n in enumerate(lengths) for t in range(-(-n // 128)) for h in range(heads)}
    real = [tuple(int(x) for x in r) for r in items if r[2] >= 0]
    assert len(real) == len(want) and set(real) == want
    for x in range(8):
        queue = items[x::8]
        queue = queue[queue[:, 2] >= 0]
        steps = _steps(kind, queue)
        end = min(len(steps), resident * 3 // 2)
        sorted_end = bool(np.all(np.diff(steps[-end:]) <= 0))
        assert sorted_end == by_cost, (x, steps[-end:])
        # before the end, and everywhere else, a chain's items follow one another
        rest = queue[:-end] if by_cost else queue
        chain = rest[:, 0].astype(np.int64) * heads + rest[:, 3]
        assert len(chain) == 0 or len(set(chain)) == 1 + int(np.sum(np.diff(chain) != 0))


def test_lists_of_grouped_heads_keep_their_order():
    """A chain that holds several query heads is walked through: a group's heads of one tile stay together."""
    items = A.schedule(A.LIST_FWD, [0, 2697, 5394, 8091], 32, 8)
    for x in range(8):
        queue = items[x::8]
        queue = queue[queue[:, 2] >= 0]
        assert np.any(np.diff(_steps(A.LIST_FWD, queue)[-96:]) > 0)
