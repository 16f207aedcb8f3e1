"""Views with more support points than a mesh workgroup stages (4096): the walks
read the row lists instead. Triangles, planes, owners and maps must equal the
oracle's, and a point must not cost far more than in a view that is staged."""
import numpy as np
import pytest

import synth
from oracle import ref

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

D0 = 6


@pytest.fixture(scope="module")
def E():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1802_07210_amd as pkg
    return pkg


def scene(kind):
    """Noise with holes, shifted by D0 columns, and the lattice step."""
    w, h, step, holes = {"long_rows": (280, 190, 2, [(60, 40, 50, 60), (200, 100, 90, 40)]),
                         # a quarter of the columns: rows of fewer than 32 points
                         "short_rows": (130, 640, 2, [(30, 0, 70, 640), (0, 300, 130, 90)]),
                         # the first rows hold nothing, some one point or two
                         "uneven_rows": (300, 260, 2, [(0, 0, 300, 90), (20, 90, 280, 30)]),
                         "every_pixel": (150, 80, 1, [(70, 30, 16, 17)])}[kind]
    rng = synth.SplitMix64(23)
    left = rng.bytes_(w * h).reshape(h, w).copy()
    for u, v, hw, hh in holes:
        left[v:v + hh, u:u + hw] = 90
    right = np.full_like(left, 90)
    right[:, :w - D0] = left[:, D0:]
    return left, right, step


@pytest.mark.parametrize("kind", ["long_rows", "short_rows", "uneven_rows", "every_pixel"])
@pytest.mark.parametrize("batched", [False, True])
def test_rows_instead_of_staged_keys(E, kind, batched):
    left, right, step = scene(kind)
    h, w = left.shape
    kw = dict(disp_max=15, candidate_stepsize=step, redun_max_dist=0, incon_min_support=0)
    t = ref.process(ref.params(**kw), left, right)
    assert len(t.ptsL) > 4096 and len(t.ptsR) > 4096
    rows = (h - 5) // step
    assert (len(t.ptsL) > 32 * rows) == (kind != "short_rows")
    dev = torch.device("cuda:0")
    L, R = torch.from_numpy(left).to(dev), torch.from_numpy(right).to(dev)
    e = E.Elas(**kw)
    oL = torch.empty((h, w), dtype=torch.int16, device=dev)
    oR = torch.empty_like(oL)
    if batched:
        e.set_batch_flags(graph=False, autotune=False)
        e.process_batch([(L, R, oL, oR)] * 2)
        get = lambda name: e.batch_intermediate(1, name)  # noqa: E731
    else:
        e.process(L, R, oL, oR)
        get = e.intermediate
    torch.cuda.synchronize()
    assert np.array_equal(get("corners"), np.concatenate([t.cornersL, t.cornersR]))
    for side, recs, planes, own in (("left", t.recL, t.planeL, t.ownerL),
                                    ("right", t.recR, t.planeR, t.ownerR)):
        assert np.array_equal(get(f"tri_{side}").reshape(-1, 9), recs)
        assert np.array_equal(get(f"plane_{side}").view(np.uint32).reshape(-1, 3),
                              planes.view(np.uint32).reshape(-1, 3))
        got = get(f"owner_{side}").reshape(h, w)
        assert np.array_equal(np.where(got == 0x7FFFFFFF, -1, got), own)
    assert np.array_equal(oL.cpu().numpy(), t.outL) and np.array_equal(oR.cpu().numpy(), t.outR)


def test_a_point_costs_about_the_same_either_way(E):
    """8 pairs of 640x480 without redundancy: about 7200 points a view (lattice
    step 5) against 3650 (step 7): 44 and 50 ns of one pair's view. Where every
    key was searched for among the row starts it was 201 and 84."""
    dev = torch.device("cuda:0")
    cfg = synth.SceneConfig(640, 480, 128, 24, 0.05, 4.0, 123.0, 2.0, 0.10, seed=3)
    p = synth.make_pair(cfg)
    L, R = torch.from_numpy(p.left).to(dev), torch.from_numpy(p.right).to(dev)
    items = [(L, R, torch.empty(L.shape, dtype=torch.int16, device=dev),
              torch.empty(L.shape, dtype=torch.int16, device=dev)) for _ in range(8)]
    cost = {}
    for step in (5, 7):
        e = E.Elas(disp_max=127, candidate_stepsize=step, redun_max_dist=0, incon_min_support=0)
        e.process(*items[0])
        torch.cuda.synchronize()
        n = e.stats()["n_support_left"]
        assert (n > 4096) == (step == 5) and n > 2500
        e.set_batch_flags(graph=False, autotune=False)
        e.set_timing(True)
        best = 1e9
        for _ in range(5):
            e.process_batch(items)
            torch.cuda.synchronize()
            best = min(best, e.timing()["mesh_ms"])
        cost[step] = best / n
    print({k: round(v * 1e6, 2) for k, v in cost.items()})
    assert cost[5] < 1.5 * cost[7]
