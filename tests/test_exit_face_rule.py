"""The tracer's exit-face rule (reciprocal products, near ties and extremes
sent to the general way) restated in numpy and compared with the general way
-- exact quotient comparisons, one IEEE division -- on the face planes of
conforming grids: the same face and the same bits of the exit distance for
random, axis-parallel, diagonal, nearly parallel and degenerate segments."""
import numpy as np
import pytest

import oracle
import synthetic

F = np.float32
X = np.longdouble  # exact 24 x 24 bit products, sums rounded to 64 bits


def dots(v):
    x, y, z = v[..., 0], v[..., 1], v[..., 2]
    return np.stack([x, y, z, x + y, x - y, x + z, x - z, y + z, y - z], axis=-1).astype(F)


def fma(a, b, c):
    return (a.astype(X) * b.astype(X) + c.astype(X)).astype(F)


def general(c, s, td, od):
    """Lowest face with the smallest exact num / den among den > 0; -1 if none."""
    num, den = np.where(s, -(c - od), c - od), np.where(s, -td, td)
    best = np.full(len(c), -1)
    bn, bd = np.zeros(len(c), F), np.ones(len(c), F)
    for f in range(4):
        better = (den[:, f] > 0) & ((best < 0) | (num[:, f].astype(np.float64) * bd < bn.astype(np.float64) * den[:, f]))
        best = np.where(better, f, best)
        bn, bd = np.where(better, num[:, f], bn), np.where(better, den[:, f], bd)
    with np.errstate(all="ignore"):
        return best, (bn / bd).astype(F)


def common(c, s, td, od, rd):
    """(taken, face, distance) of the reciprocal rule."""
    with np.errstate(all="ignore"):
        num = (c - od).astype(F)
        q = np.where(s ^ np.signbit(rd), F(np.inf), (num * rd).astype(F))
        b = np.fmin(np.fmin(q[:, 0], q[:, 1]), np.fmin(q[:, 2], q[:, 3]))
        m = q <= fma(np.abs(b), np.full_like(b, 2.0 ** -20), b)[:, None]
        taken = (m.sum(axis=1) <= 1) & (b > F(2.0 ** -40))
        face = np.where(m[:, 3], 3, np.where(m[:, 2], 2, np.where(m[:, 1], 1, 0)))
        at = np.arange(len(c))
        n, r, d = num[at, face], rd[at, face], td[at, face]
        q1 = fma(fma(-b, d, n), r, b)
        return taken, face, fma(fma(-q1, d, n), r, q1)


def directions(kind, k, rng):
    v = rng.normal(size=(k, 3))
    v /= np.linalg.norm(v, axis=1)[:, None]
    if kind == "axes":
        v = np.eye(3)[rng.integers(0, 3, k)] * rng.choice([-1, 1], (k, 1))
    elif kind == "diagonals":
        v = rng.choice([-1.0, 0.0, 1.0], (k, 3)) * 0.7071068
    elif kind == "grazing":  # one plane direction's product nearly vanishes
        v[:, 1] = v[:, 0] * (1 + rng.choice([0.0, 1e-7, -1e-7, 1e-6], k))
    elif kind == "tiny":
        v = rng.choice([1e-38, 1e-30, 1e-20, 1e-13, 2.0 ** -40, 1.0, -1.0, 0.0], (k, 3))
    return v.astype(F)


@pytest.mark.parametrize("kind", ["random", "axes", "diagonals", "grazing", "tiny"])
@pytest.mark.parametrize("scale", [2.0 ** 20, 1.0])  # lattice units (compact records), world units
def test_reciprocal_rule_equals_general_way(kind, scale):
    sc = synthetic.scene("blobs_adaptive")
    g = oracle.leb_build(sc["density_fn"](), 32, sc["camera"], sc["build"])
    e = g.export()
    rng = np.random.default_rng(7)
    k = 200000
    cell = rng.integers(0, len(e["ids"]), k)
    verts = e["verts"][cell].astype(np.float64) / 2.0 ** 20
    w = rng.dirichlet([1.0] * 4, k)
    w[: k // 4] = np.eye(4)[rng.integers(0, 4, k // 4)]  # origins at vertices: ties at zero
    o = (w[:, :, None] * verts).sum(axis=1).astype(F)
    d = directions(kind, k, rng)
    codes, offs = e["codes"][cell].astype(np.int64), e["offsets"][cell].astype(np.int64)
    N, s = codes >> 1, (codes & 1).astype(bool)
    c = (np.where(s, -offs, offs) * (scale / 2.0 ** 20)).astype(F)
    td9, od9 = dots(d), dots((o * F(scale)).astype(F))
    tiny = (d == 0).all(axis=1) | ((td9 != 0) & ~((td9 <= -F(2.0 ** -40)) | (td9 >= F(2.0 ** -40)))).any(axis=1)
    with np.errstate(all="ignore"):
        rd9 = np.where(tiny[:, None], F(0), np.where(td9 == 0, F(np.nan), F(1) / td9)).astype(F)
    td, od, rd = (np.take_along_axis(x, N, axis=1) for x in (td9, od9, rd9))
    face, te = general(c, s, td, od)
    taken, f2, t2 = common(c, s, td, od, rd)
    assert not taken[tiny].any() and not taken[face < 0].any()
    assert (kind == "tiny") or taken.mean() > 0.25  # the rule is worth having
    assert (f2[taken] == face[taken]).all()
    assert (t2[taken].view(np.uint32) == te[taken].view(np.uint32)).all()


@pytest.mark.parametrize("kind", ["random", "axes", "diagonals", "grazing", "tiny"])
def test_voxel_rule_equals_division_of_every_axis(kind):
    """The voxel walk's form of the rule: the axis with the smallest rounded
    distance (plane - o) / d, the lowest axis on ties, and that distance."""
    rng = np.random.default_rng(9)
    k, n = 300000, 64
    cell = rng.integers(0, n, (k, 3))
    o = ((cell + rng.random((k, 3))) / n).astype(F)
    o[: k // 3] = (cell[: k // 3] / n).astype(F)  # on voxel faces, edges and corners
    d = directions(kind, k, rng)
    num = ((cell + (d > 0)) / F(n)).astype(F) - o
    td9 = dots(d)
    tiny = (d == 0).all(axis=1) | ((td9 != 0) & ~((td9 <= -F(2.0 ** -40)) | (td9 >= F(2.0 ** -40)))).any(axis=1)
    with np.errstate(all="ignore"):
        tf = (num / d).astype(F)
        best, bt = np.full(k, -1), np.zeros(k, F)
        for a in range(3):
            better = (d[:, a] != 0) & ((best < 0) | (tf[:, a] < bt))
            best, bt = np.where(better, a, best), np.where(better, tf[:, a], bt)
        r = np.where(tiny[:, None], F(0), np.where(d == 0, F(np.nan), F(1) / d)).astype(F)
        q = (num * r).astype(F)
        b = np.fmin(np.fmin(q[:, 0], q[:, 1]), q[:, 2])
        m = q <= fma(np.abs(b), np.full_like(b, 2.0 ** -20), b)[:, None]
        taken = (m.sum(axis=1) <= 1) & (b > F(2.0 ** -40))
        axis = np.where(m[:, 2], 2, np.where(m[:, 1], 1, 0))
        at = np.arange(k)
        q1 = fma(fma(-b, d[at, axis], num[at, axis]), r[at, axis], b)
        te = fma(fma(-q1, d[at, axis], num[at, axis]), r[at, axis], q1)
    assert not taken[tiny].any() and not taken[best < 0].any()
    assert (kind == "tiny") or taken.mean() > 0.25
    assert (axis[taken] == best[taken]).all()
    assert (te[taken].view(np.uint32) == bt[taken].view(np.uint32)).all()
