"""Point location by folding coordinates, restated in Python and compared with
bisecting the tet's vertices: the same path to every depth, for both tie
rules, points on planes, edges and vertices, and (in doubles) for every kind
of coordinate that the folding is taken for."""
import itertools
from fractions import Fraction

import numpy as np
import pytest

PERMS = [(0, 1, 2), (0, 2, 1), (1, 0, 2), (1, 2, 0), (2, 0, 1), (2, 1, 0)]
S = 1 << 20


def fold(f0, f1, f2, s, dmax, h, above):
    over = (lambda a, b: a >= b) if above else (lambda a, b: a > b)
    for _ in range(0, dmax, 3):
        b1 = over(f0 + f2, s)
        b2 = over((f2 if b1 else f0) + f1, s)
        p = (f2 if b2 else f1) if b1 else (f1 if b2 else f0)
        b3, r0 = over(p, s - p), s - f0
        f1, f2 = (s - f1 if b2 else f2) if b1 else (r0 if b2 else f1), r0 if b1 else f2
        f0, s, h = s - p if b3 else p, s / 2, 8 * h + 4 * b1 + 2 * b2 + b3
    return h >> (-dmax % 3)


def bisect(p, root, dmax, above):
    """Bisections of the root's vertices; p's type carries the arithmetic."""
    v = [[0, 0, 0]]
    for a in PERMS[root]:
        v.append([S if i == a else x for i, x in enumerate(v[-1])])
    v = [[Fraction(x) for x in w] for w in v]
    h = 8 + root
    for d in range(dmax):
        k = 3 - d % 3
        m = [(a + b) / 2 for a, b in zip(v[0], v[k])]
        a, b = (v[j] for j in range(1, 4) if j != k)
        x, y = [s - t for s, t in zip(a, m)], [s - t for s, t in zip(b, m)]
        n = [x[1] * y[2] - x[2] * y[1], x[2] * y[0] - x[0] * y[2], x[0] * y[1] - x[1] * y[0]]
        if sum(c * (s - t) for c, s, t in zip(n, v[0], m)) < 0:
            n = [-c for c in n]
        side = type(p[0])(0)
        for c, q, t in zip(n, p, m):
            if c:
                t = q - type(q)(t)
                side = side + (t if c > 0 else -t)
        first = side > 0 if above else side >= 0
        v = [m if j == k else (v[j] if first or j > k else v[j + 1]) for j in range(4)]
        h = 2 * h + (not first)
    return h


def roots_of(p):
    return [(r, [p[a] for a in o]) for r, o in enumerate(PERMS) if p[o[0]] >= p[o[1]] >= p[o[2]]]


@pytest.mark.parametrize("above", [False, True])
@pytest.mark.parametrize("den", [1, 3, 64, 1000003])
def test_folding_is_bisection(den, above):
    rng = np.random.default_rng(den)
    pts = [[Fraction(int(x), den) * (S // 64) for x in rng.integers(0, 64 * den + 1, 3)] for _ in range(60)]
    pts += [[Fraction(c * S, 2) for c in q] for q in itertools.product(range(3), repeat=3)]
    for p in pts:
        for r, f in roots_of(p):
            for d in (0, 1, 2, 3, 10, 20):
                assert fold(*f, Fraction(S), d, 8 + r, above) == bisect(p, r, d, above)


def test_folding_in_doubles_is_bisection_in_doubles():
    """Coordinates 0 or at least 2^-29: both are exact, so they agree to the
    last plane, also where sums differ from it by one unit in the last place."""
    rng = np.random.default_rng(5)
    pts = []
    for k in range(150):
        p = rng.random(3).astype(np.float32)
        p[k % 3] = np.float32(2.0) ** np.float32(-rng.integers(1, 30)) * np.float32(1 + rng.random())
        if k % 4 == 0:  # on or one ulp off the plane a + b = 1
            p[(k + 1) % 3] = np.float32(1) - p[k % 3]
        if k % 8 == 0:
            p[(k + 1) % 3] = np.nextafter(p[(k + 1) % 3], np.float32(0))
        if k % 5 == 0:
            p[(k + 2) % 3] = rng.integers(0, 2)
        pts.append(np.clip(p, 0, 1))
    for p in pts:
        q = [float(x) * S for x in p]
        assert all(x == 0 or x >= 2.0 ** -9 for x in q)
        for r, f in roots_of(q):
            want = bisect([Fraction(x) for x in q], r, 57, False)
            assert fold(*f, float(S), 57, 8 + r, False) == want
            assert bisect(q, r, 57, False) == want
