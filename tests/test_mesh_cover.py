"""The sums by which the device mesh's triangles are checked (doubled area and
first moments against the image rectangle's, modulo 2^32), on the oracle's
meshes: a mesh passes, one with a planted mistake does not."""
import random

import numpy as np
import pytest

from oracle import ref


def covers(recs, w, h):
    """As mesh_covers over the raster records."""
    a = au = av = 0
    for r in recs:
        u, v = [int(x) for x in r[0::3]], [int(x) for x in r[1::3]]
        d = abs((u[1] - u[0]) * (v[2] - v[0]) - (u[2] - u[0]) * (v[1] - v[0]))
        a, au, av = a + d, au + d * sum(u), av + d * sum(v)
    x, y, m = w - 1, h - 1, 1 << 32
    return (a % m, au % m, av % m) == (2 * x * y % m, 3 * x * x * y % m, 3 * x * y * y % m)


def mesh(rng, w, h, step, n):
    pts = [(u, v) for v in range(4 + step, h - 4, step) for u in range(4 + step, w - 4, step)]
    pts = sorted(rng.sample(pts, min(n, len(pts))), key=lambda p: (p[1], p[0]))
    uvd = np.array([(0, 0, 1), (w - 1, 0, 1), (0, h - 1, 1), (w - 1, h - 1, 1)] +
                   [(u, v, 3) for u, v in pts], np.int32)
    return ref.canonical(uvd, ref.delaunay(uvd[:, :2]))


@pytest.mark.parametrize("w,h,step,n", [(60, 40, 5, 12), (160, 120, 5, 90), (131, 77, 2, 60),
                                        (4096, 4096, 97, 80), (4095, 211, 13, 40), (40, 40, 10, 1)])
def test_sums_tell_a_mesh_from_one_with_a_mistake(w, h, step, n):
    rng = random.Random(w * h + n)
    recs = [tuple(r) for r in mesh(rng, w, h, step, n).tolist()]
    assert covers(recs, w, h)
    for _ in range(40):
        i, j = rng.sample(range(len(recs)), 2)
        assert not covers(recs[:i] + recs[i + 1:], w, h)              # one missing
        bad = list(recs)
        bad[i] = recs[j]                                              # one twice, one missing
        assert not covers(bad, w, h)
        r = list(recs[i])
        k = rng.randrange(3)
        other = recs[j][3 * rng.randrange(3):][:3]
        if tuple(r[3 * k:3 * k + 2]) != tuple(other[:2]):
            r[3 * k:3 * k + 3] = other                                # a wrong vertex
            bad[i] = tuple(r)
            assert not covers(bad, w, h)
