"""A device mesh that gives up in one view only: that view has no plane prior,
the other view's prior is the oracle's, and the frame is reported as failed.

The walk limit (a test hook) is set between what the two views need; the need
of a view, the most searches any of its points makes in one direction, is
worked out here from the oracle's triangles."""
import numpy as np
import pytest

import synth
from oracle import ref

W, H, D = 160, 120, 48
KW = dict(disp_max=D - 1)


def searches_needed(pts, recs):
    """Most searches of one walk: its triangles, and one more to meet the
    smaller list point that ends it (none after a top corner)."""
    listed = {(int(v), int(u)) for u, v, _ in pts}
    own = {}
    for r in recs.tolist():
        verts = [(r[1], r[0]), (r[4], r[3]), (r[7], r[6])]
        mine = sorted(x for x in verts if x in listed)
        if mine:
            own.setdefault(mine[0], []).append([x for x in verts if x != mine[0]])
    below = sorted(listed) + [(H - 1, 0), (H - 1, W - 1)]
    most = 0
    for p, tris in own.items():
        def cross(a, b):
            return (a[1] - p[1]) * (b[0] - p[0]) - (a[0] - p[0]) * (b[1] - p[1])
        first = None  # the smallest circle tangent to p's row; the first in turning order on ties
        for c in below:
            n, d = (c[1] - p[1]) ** 2 + (c[0] - p[0]) ** 2, c[0] - p[0]
            if d <= 0:
                continue
            if first is None or n * first[2] < first[1] * d or \
                    (n * first[2] == first[1] * d and cross(c, first[0]) > 0):
                first = (c, n, d)
        for sgn in (1, -1):
            side = [t for t in tris if any(sgn * cross(first[0], x) > 0 for x in t)]
            top = any(x[0] == 0 for t in side for x in t)
            most = max(most, len(side) + (0 if top else 1))
    return most


def scene(seed):
    cfg = synth.SceneConfig(W, H, D, 6, 0.05, 4.0, D - 5.0, 2.0, 0.15, patch=24, seed=seed)
    return synth.make_pair(cfg)


def oracle(seed):
    p = scene(seed)
    t = ref.process(ref.params(**KW), p.left, p.right)
    return p, t, searches_needed(t.ptsL, t.recL), searches_needed(t.ptsR, t.recR)


# seeds by the view that needs more searches
LEFT_NEEDS_MORE, RIGHT_NEEDS_MORE = [6, 7, 21], [0, 9, 17]


@pytest.mark.parametrize("seed,left_more", [(s, True) for s in LEFT_NEEDS_MORE] +
                         [(s, False) for s in RIGHT_NEEDS_MORE])
def test_scenes_differ_as_stated(seed, left_more):
    _, t, needL, needR = oracle(seed)
    assert len(t.ptsL) > 10 and len(t.ptsR) > 10
    assert (needL > needR) if left_more else (needR > needL)


@pytest.mark.gpu
@pytest.mark.parametrize("batched", [False, True])
@pytest.mark.parametrize("seed", LEFT_NEEDS_MORE + RIGHT_NEEDS_MORE)
def test_only_the_failing_view_loses_its_prior(seed, batched):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1802_07210_amd as E

    dev = torch.device("cuda:0")
    p, t, needL, needR = oracle(seed)
    other = scene(seed + 100)
    e = E.Elas(**KW)
    e.set_batch_flags(graph=True, autotune=False)

    def call(q):
        L, R = torch.from_numpy(q.left).to(dev), torch.from_numpy(q.right).to(dev)
        oL = torch.empty((H, W), dtype=torch.int16, device=dev)
        oR = torch.empty_like(oL)
        if batched:
            e.process_batch([(L, R, oL, oR)])
        else:
            e.process(L, R, oL, oR)
        torch.cuda.synchronize()

    call(other)  # another frame's triangles are in the buffers
    e.set_mesh_round_limit(min(needL, needR))
    call(p)
    get = (lambda name: e.batch_intermediate(0, name)) if batched else e.intermediate
    for side, fails, own, dpl, n in (("left", needL > needR, t.ownerL, t.dplaneL, len(t.recL)),
                                     ("right", needR > needL, t.ownerR, t.dplaneR, len(t.recR))):
        owner = get(f"owner_{side}").reshape(H, W)
        plane = get(f"dplane_{side}").reshape(H, W)
        if fails:
            assert (owner == 0x7FFFFFFF).all() and (plane == -1).all()
            assert get(f"tri_{side}").size == 0
        else:
            assert np.array_equal(np.where(owner == 0x7FFFFFFF, -1, owner), own)
            assert np.array_equal(plane, dpl)
            assert get(f"tri_{side}").size == 9 * n
    with pytest.raises(E.ElasError, match="ELAS_ERR_INTERNAL"):
        call(p)
    e.set_mesh_round_limit(32000)
    call(p)
    for side, own in (("left", t.ownerL), ("right", t.ownerR)):
        owner = get(f"owner_{side}").reshape(H, W)
        assert np.array_equal(np.where(owner == 0x7FFFFFFF, -1, owner), own)
