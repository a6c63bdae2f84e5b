"""Host replay of the left-looking launch's schedule (qd): workgroups take the
next column from a counter, wait for each earlier column in turn, and finish
theirs.  It must end whatever number of workgroups is on the card at a time
and however their steps interleave, with every column taken once and its
projections in order.  Columns dealt by workgroup number stall as soon as
some workgroup cannot start.

No arithmetic: a column's state is the number of its projections so far.
"""
import random

import pytest


def replay(ncols, groups, resident, seed, dealt):
    """Columns finished, or None when no workgroup on the card can go on."""
    r = random.Random(seed)
    order = list(range(groups))  # the order in which they get their place
    r.shuffle(order)
    card, counter = [], 0
    seen = [[] for _ in range(ncols)]
    done = [False] * ncols

    def start(g):
        return dict(g=g, c=None, last=-1)

    while order or card:
        while order and len(card) < resident:
            card.append(start(order.pop()))
        moved = False
        for w in r.sample(card, len(card)):
            if w["c"] is None:  # the next column
                if dealt:
                    w["c"] = w["g"] if w["last"] < 0 else w["last"] + groups
                elif w["last"] == ncols - 1:
                    w["c"] = ncols
                else:
                    w["c"], counter = counter, counter + 1
                moved = True
                if w["c"] >= ncols:
                    card.remove(w)
                    break
                w["k"] = 0
            elif w["k"] == w["c"]:
                done[w["c"]], w["last"], w["c"], moved = True, w["c"], None, True
            elif done[w["k"]]:
                seen[w["c"]].append(w["k"])
                w["k"] += 1
                moved = True
        if not moved:
            return None
    assert all(done) and all(s == list(range(c)) for c, s in enumerate(seen))
    return sum(done)


@pytest.mark.parametrize("ncols,groups", [(1, 1), (2, 2), (9, 9), (30, 8), (61, 20)])
@pytest.mark.parametrize("seed", range(4))
def test_ends_with_any_number_of_workgroups_on_the_card(ncols, groups, seed):
    for resident in {1, 2, (groups + 1) // 2, groups}:
        assert replay(ncols, groups, resident, seed, False) == ncols


def test_columns_dealt_by_number_need_all_of_them():
    assert replay(30, 8, 8, 0, True) == 30
    assert any(replay(30, 8, 4, seed, True) is None for seed in range(4))
