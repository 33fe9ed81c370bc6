"""The build's rule for edges whose midpoints can be vertices, restated in
Python and compared with the bisection tree: every tet around an edge bisects
it at one depth, the depth that the rule gives for each of its tets."""
import itertools

import pytest

# depth at which a tet of tag 3, 2, 1 bisects each of its edges, less its own
LEVELS = {3: {(0, 1): 2, (0, 2): 1, (0, 3): 0, (1, 2): 2, (1, 3): 1, (2, 3): 2},
          2: {(0, 1): 1, (0, 2): 0, (0, 3): 2, (1, 2): 1, (1, 3): 2, (2, 3): 2},
          1: {(0, 1): 0, (0, 2): 2, (0, 3): 1, (1, 2): 2, (1, 3): 1, (2, 3): 3}}
WORDS = {3: 0x3F3F1604, 2: 0x3F3F0B02, 1: 0x3F1F1501}  # a byte of edge bits per number of levels below
EDGES = list(itertools.combinations(range(4), 2))


@pytest.mark.parametrize("tag", [3, 2, 1])
def test_words(tag):
    for s in range(4):
        bits = sum(1 << k for k, e in enumerate(EDGES) if LEVELS[tag][e] <= s)
        assert (WORDS[tag] >> (8 * s)) & 0xFF == bits


def test_levels_of_the_bisection_tree():
    side, depth = 1 << 8, 13
    tets = []
    for order in itertools.permutations(range(3)):
        v = [(0, 0, 0)]
        for a in order:
            v.append(tuple(side if i == a else x for i, x in enumerate(v[-1])))
        tets.append(v)
    rule, seen = {}, {}
    for d in range(depth):
        k, below = 3 - d % 3, []
        for v in tets:
            for i, j in EDGES:
                e = frozenset((v[i], v[j]))
                assert rule.setdefault(e, d + LEVELS[k][i, j]) == d + LEVELS[k][i, j]
            m = tuple((a + b) // 2 for a, b in zip(v[0], v[k]))
            assert rule[frozenset((v[0], v[k]))] == d
            assert seen.setdefault(m, frozenset((v[0], v[k]))) == frozenset((v[0], v[k]))  # one edge per midpoint
            below.append([m if j == k else v[j] for j in range(4)])
            below.append([v[j + 1] if j < k else (m if j == k else v[j]) for j in range(4)])
        tets = below
