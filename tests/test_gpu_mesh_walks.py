"""The device mesh at the places where its walks can go wrong, against the
oracle: a point with more neighbours than its chain holds (the overflow list),
clusters with more points around one than the listed box holds, and large
empty parts whose circles reach far beyond the box. Triangles, planes and
owners must equal the oracle's in single and batched calls."""
import numpy as np
import pytest

import synth
from oracle import ref

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

W, H, STEP, D0 = 520, 440, 10, 9


@pytest.fixture(scope="module")
def E():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1802_07210_amd as pkg
    return pkg


def lattice_points(kind):
    us, vs = range(40, W - 20, STEP), range(20, H - 20, STEP)
    every = [(u, v) for v in vs for u in us]
    r2 = {p: (p[0] - 270) ** 2 + (p[1] - 220) ** 2 for p in every}
    if kind == "hub":        # one point inside a ring: all of the ring are its neighbours
        return [p for p in every if p == (270, 220) or 185 ** 2 <= r2[p] < 196 ** 2]
    if kind == "low_hub":    # most neighbours on one side of the first one
        return [p for p in every if p == (270, 60) or (170 ** 2 <= r2[p] < 182 ** 2 and p[1] > 80)]
    if kind == "cluster":    # dense block, few points elsewhere
        return [p for p in every if (abs(p[0] - 120) <= 70 and abs(p[1] - 100) <= 70) or
                p in ((340, 40), (450, 360), (60, 370))]
    return [p for p in every if p[0] in (40, 50, 450) or p[1] in (20, 410)]  # "frame"


def scene(kind):
    rng = synth.SplitMix64(17)
    left = np.full((H, W), 90, np.uint8)
    for u, v in lattice_points(kind):
        left[v - 4:v + 5, u - 4:u + 5] = rng.bytes_(81).reshape(9, 9)
    right = np.full_like(left, 90)
    right[:, :W - D0] = left[:, D0:]
    return left, right


@pytest.mark.parametrize("kind", ["hub", "low_hub", "cluster", "frame"])
@pytest.mark.parametrize("batched", [False, True])
def test_walks(E, kind, batched):
    left, right = scene(kind)
    kw = dict(disp_max=31, candidate_stepsize=STEP, redun_max_dist=0, incon_min_support=0)
    t = ref.process(ref.params(**kw), left, right)
    assert len(t.ptsL) >= 15
    dev = torch.device("cuda:0")
    L, R = torch.from_numpy(left).to(dev), torch.from_numpy(right).to(dev)
    e = E.Elas(**kw)
    oL = torch.empty((H, W), dtype=torch.int16, device=dev)
    oR = torch.empty_like(oL)
    if batched:
        e.set_batch_flags(graph=False, autotune=False)
        e.process_batch([(L, R, oL, oR)] * 2)
        get = lambda name: e.batch_intermediate(1, name)  # noqa: E731
    else:
        e.process(L, R, oL, oR)
        get = e.intermediate
    torch.cuda.synchronize()
    for side, recs, planes, own in (("left", t.recL, t.planeL, t.ownerL),
                                    ("right", t.recR, t.planeR, t.ownerR)):
        assert np.array_equal(get(f"tri_{side}").reshape(-1, 9), recs)
        assert np.array_equal(get(f"plane_{side}").view(np.uint32).reshape(-1, 3),
                              planes.view(np.uint32).reshape(-1, 3))
        got = get(f"owner_{side}").reshape(H, W)
        assert np.array_equal(np.where(got == 0x7FFFFFFF, -1, got), own)
    assert np.array_equal(oL.cpu().numpy(), t.outL) and np.array_equal(oR.cpu().numpy(), t.outR)
