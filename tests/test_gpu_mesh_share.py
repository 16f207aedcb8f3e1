"""The mesh's workgroups of a batch follow the points of all its frames: few
small frames must still spread over the chip, and a batch's maps do not depend
on how many frames share the call."""
import numpy as np
import pytest

import synth
from oracle import ref

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def E():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1802_07210_amd as pkg
    return pkg


def pair(w, h, D, seed):
    cfg = synth.SceneConfig(w, h, D, 5, 0.05, 4.0, D - 5.0, 2.0, 0.10, patch=24, seed=seed)
    return synth.make_pair(cfg)


def items_of(E, pairs, n):
    dev = torch.device("cuda:0")
    out = []
    for i in range(n):
        p = pairs[i % len(pairs)]
        L, R = torch.from_numpy(p.left).to(dev), torch.from_numpy(p.right).to(dev)
        oL = torch.empty(L.shape, dtype=torch.int16, device=dev)
        out.append((L, R, oL, torch.empty_like(oL)))
    return out


# 1 and 2 frames take the least share (72 lattice points), 96 of 97x61 and 40 of
# 320x240 one between, 9 of 1280x720 the largest (384)
@pytest.mark.parametrize("w,h,D,n", [(97, 61, 24, 1), (200, 120, 32, 2), (97, 61, 24, 96),
                                     (320, 240, 64, 40), (1280, 720, 192, 9)])
def test_batches_of_any_share_match_the_oracle(E, w, h, D, n):
    pairs = [pair(w, h, D, s) for s in range(2)]
    t = [ref.process(ref.params(disp_max=D - 1), p.left, p.right) for p in pairs]
    e = E.Elas(disp_max=D - 1)
    e.set_batch_flags(graph=True, autotune=False)
    items = items_of(E, pairs, n)
    for rep in range(2):
        e.process_batch(items)
    torch.cuda.synchronize()
    for i in {0, 1 % n, n // 2, n - 1}:
        r = t[i % 2]
        assert np.array_equal(e.batch_intermediate(i, "tri_left").reshape(-1, 9), r.recL)
        assert np.array_equal(e.batch_intermediate(i, "tri_right").reshape(-1, 9), r.recR)
        assert np.array_equal(items[i][2].cpu().numpy(), r.outL)
        assert np.array_equal(items[i][3].cpu().numpy(), r.outR)


def test_small_frames_spread_over_the_chip(E):
    """The mesh of 64 pairs of 128x128 against that of a plain call: its points
    fit the chip's wavefronts one or two each, where the plain call takes two
    wavefronts a point (27 and 18 us; 43 with 384 lattice points to a
    workgroup)."""
    pairs = [pair(128, 128, 32, 1)]
    e = E.Elas(disp_max=31)
    e.set_batch_flags(graph=False, autotune=False)
    e.set_timing(True)
    items = items_of(E, pairs, 64)
    best = {}
    for name, call in (("plain", lambda: e.process(*items[0])),
                       ("batch", lambda: e.process_batch(items))):
        ms = []
        for _ in range(8):
            call()
            torch.cuda.synchronize()
            ms.append(e.timing()["mesh_ms"])
        best[name] = min(ms)
    print({k: round(v * 1e3, 1) for k, v in best.items()})
    assert best["batch"] < 1.9 * best["plain"]
