"""The local-index remap in the layout that the walk reads: a byte for each order
of the entry face's slots (three 2-bit fields), exit slot and rank of the
neighbour's new vertex.  The library numbers an element's vertices by ascending
node id, so the byte holds the ranks of the slots among the neighbour's nodes."""

import itertools

import pytest

from test_mesh_edge_max_cpu import probe_lib


@pytest.fixture(scope="module")
def remap():
    return probe_lib().probe_walk_remap


@pytest.mark.parametrize("k", [0, 1, 2])
@pytest.mark.parametrize("back", [0, 1, 2, 3])
def test_walk_reads_the_ranks_in_the_neighbour(remap, k, back):
    for perm in itertools.permutations(range(4)):  # ranks of slots 0, 1, 2 and of v
        # Node 10 p has rank p; the new vertex goes between its neighbours in rank.
        shared = [10 * p for s, p in enumerate(perm) if s != k]
        new = sorted(shared)[back] - 1 if back < 3 else 100
        nodes = sorted(shared + [new])
        slots = [10 * perm[3] if s == k else 10 * perm[s] for s in range(3)]
        loc = sum(p << (2 * s) for s, p in enumerate(perm[:3]))
        assert nodes.index(new) == back
        assert remap(loc, k, back) == sum(nodes.index(x) << (2 * s) for s, x in enumerate(slots))
