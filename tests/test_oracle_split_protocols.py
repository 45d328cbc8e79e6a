"""Exhaustive interleaving checks of the protocols in which many workgroups act
as one endpoint (oracle/protocol_split.py; CPU only): rings whose ends are split
over teams, and ping-pong's counter tree.  Each accepted configuration is
explored completely; each planted mistake must be caught."""
import pytest

from oracle import protocol_split as ps
from oracle.protocol_kernels import Violation

# P, E, sizes, teams, members of a team, messages and bytes of a group, byte counter
SPLIT = [
    (4, 3, [2, 1, 2], 2, 1, 1, 9, 0),
    (4, 3, [2, 2, 1, 2], 1, 2, 1, 9, 0),
    (3, 2, [2, 1, 2], 2, 2, 1, 9, 0),
    (4, 4, [1, 1, 2, 1], 2, 2, 2, 2, 0),         # groups of two messages
    (5, 3, [0, 3, 1, 2], 2, 2, 1, 9, 0),         # an empty message, shares that are none
    (4, 3, [1, 2, 1, 2, 1], 2, 1, 2, 2, 3),      # a ring that starts in its middle
    (4, 2, [2, 2, 2], 2, 2, 1, 9, 3),
    (3, 3, [1, 3, 1], 3, 1, 1, 9, 1),            # a message as large as the ring
]


@pytest.mark.parametrize("cfg", SPLIT)
def test_split_ring_accepts(cfg):
    assert ps.explore_split(*cfg) > 200


def _caught(cfg, bug):
    try:
        ps.explore_split(*cfg, ps.Bug(**{bug: True}))
    except Violation as e:
        return str(e)
    return None


@pytest.mark.parametrize("bug,shared", [
    ("publish_without_others", True), ("release_without_others", True),
    ("waits_without_share", True), ("publish_out_of_turn", False),
    ("release_out_of_turn", False), ("entries_only", False), ("stale_base", False)])
def test_split_ring_catches(bug, shared):
    cfgs = [c for c in SPLIT if not shared or c[4] > 1]
    found = [_caught(c, bug) for c in cfgs]
    # in every configuration in which the mistake can show, and in at least two
    assert sum(f is not None for f in found) >= 2, (bug, found)
    if bug == "waits_without_share":
        assert any(f and f.startswith("deadlock") for f in found)


def test_groups_are_cut_alike_and_fit():
    assert ps.groups_of([5, 1, 1, 1, 9, 0, 0], 8, 3, 4) == [(0, 1), (1, 4), (4, 5), (5, 7)]
    assert ps.groups_of([1, 1, 1], 2, 16, 100) == [(0, 2), (2, 3)]


@pytest.mark.parametrize("W,G,reps", [(2, 1, 2), (2, 2, 2), (3, 2, 1), (3, 2, 2), (4, 2, 1), (4, 3, 1)])
def test_counter_tree_accepts(W, G, reps):
    assert ps.explore_tree(W, G, reps) > 100


@pytest.mark.parametrize("bug", ["flags_by_neighbours", "count_before_copy"])
@pytest.mark.parametrize("W,G,reps", [(3, 2, 2), (4, 2, 1)])
def test_counter_tree_catches(W, G, reps, bug):
    with pytest.raises(Violation):
        ps.explore_tree(W, G, reps, ps.Bug(**{bug: True}))
