"""The facts the device mesh's walks rely on, checked on the CPU against the
oracle's triangulation: every list point's own triangles, found from its first
neighbour (the smallest circle tangent to its row from below) by stepping to
the neighbour with the smallest circle on either side, plus the one triangle on
the top image side, are the canonical mesh. Co-circular points go to the
(v, u)-smallest one if it is smaller than the walking point, else to the first
in walking order."""
import random

import numpy as np
import pytest

from oracle import ref


def walk_mesh(points, w, h):
    """Triangles as sorted (v, u) triples."""
    pts = sorted((v, u) for u, v, _ in points)
    corners = [(0, 0), (0, w - 1), (h - 1, 0), (h - 1, w - 1)]
    everything, top = pts + corners, set(corners[:2])

    def search(p, e, f, sgn, tangent=False):
        best = None
        for c in everything:
            dx, dy = c[1] - p[1], c[0] - p[0]
            D = f[0] * dy - f[1] * dx
            if D <= 0:
                continue
            N = dx * (dx - e[0]) + dy * (dy - e[1])
            if best is None or N * best[2] < best[1] * D:
                best = (c, N, D)
            elif N * best[2] == best[1] * D and not tangent:
                cur = best[0]
                if min(c, cur) < p:
                    take = c < cur
                else:
                    take = sgn * (dx * (cur[0] - p[0]) - dy * (cur[1] - p[1])) > 0
                if take:
                    best = (c, N, D)
        return best[0]

    tris = []
    for p in pts:
        q0 = search(p, (0, 0), (1, 0), 1, tangent=True)
        for sgn in (1, -1):
            q = q0
            while True:
                e = (q[1] - p[1], q[0] - p[0])
                r = search(p, e, (sgn * e[0], sgn * e[1]), sgn)
                if r < p and r not in top:
                    break
                tris.append(tuple(sorted((p, q, r))))
                if r in top:
                    break
                q = r
    apex = search(corners[0], (w - 1, 0), (w - 1, 0), 1)
    tris.append(tuple(sorted((corners[0], corners[1], apex))))
    return sorted(tris)


@pytest.mark.parametrize("seed", range(12))
def test_walks_give_the_canonical_mesh(seed):
    rng = random.Random(seed)
    for _ in range(8):
        w, h = rng.randint(20, 160), rng.randint(20, 120)
        step = rng.choice([1, 2, 5, 5, 10])
        lattice = [(u, v) for v in range(4 + step, h - 4, step)
                   for u in range(4 + step, w - 4, step)]
        if not lattice:
            continue
        pts = rng.sample(lattice, rng.randint(1, min(len(lattice), 60)))
        shape = rng.random()
        if shape < 0.25:    # columns off the lattice, as seen from the right view
            pts = [(max(1, u - rng.randint(0, 3)), v) for u, v in pts]
        elif shape < 0.35:  # one row
            pts = [p for p in pts if p[1] == pts[0][1]]
        elif shape < 0.45:  # one column
            pts = [p for p in pts if p[0] == pts[0][0]]
        pts = sorted(set(pts), key=lambda p: (p[1], p[0]))
        corners = [(0, 0), (w - 1, 0), (0, h - 1), (w - 1, h - 1)]
        uv = np.array(corners + pts, np.int32)
        uvd = np.concatenate([uv, np.full((len(uv), 1), 3, np.int32)], axis=1)
        recs = ref.canonical(uvd, ref.delaunay(uv))
        want = [tuple((r[3 * k + 1], r[3 * k]) for k in range(3))
                for r in np.asarray(recs).reshape(-1, 9).tolist()]
        assert walk_mesh([(u, v, 3) for u, v in pts], w, h) == want
