"""Dense matching with the check in the same kernel at the row widths where it
can go wrong: below, at and above a 64-pixel piece, the staging steps of 768
and 1536 columns (256 and 512 threads), the widths where a batch changes the
threads per row, and the last width it takes (2112 columns of gradient
descriptors; wider rows go through the two separate kernels, census ones above
3840). Everything is compared with the CPU oracle exactly."""
import numpy as np
import pytest

import synth
from oracle import ref

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CENSUS = dict(descriptor=1, census_support_window=9, census_dense_window=5, median_window=3)


def pair(w, h, D):
    return synth.make_pair(synth.SceneConfig(w, h, D, 5, 0.05, 2.0, D - 3.0, 2.0, 0.05, seed=w))


def check(e, t, oL, oR):
    assert np.array_equal(oL, t.outL) and np.array_equal(oR, t.outR)
    assert np.array_equal(e.intermediate("raw_left").reshape(t.rawL.shape), t.rawL)
    assert np.array_equal(e.intermediate("raw_right").reshape(t.rawR.shape), t.rawR)


@pytest.mark.parametrize("kw", [{}, CENSUS], ids=["gradient", "census_median"])
@pytest.mark.parametrize("w", [13, 63, 64, 65, 128, 191, 705, 769, 1537, 2112, 2113, 3905])
def test_fused_match_widths(w, kw):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1802_07210_amd as E
    D = 8 if w < 128 else 24
    p, kw = pair(w, 31, D), dict(disp_max=D - 1, **kw)
    dev = torch.device("cuda:0")
    e = E.Elas(**kw)
    oL, oR = e.process(torch.from_numpy(p.left).to(dev), torch.from_numpy(p.right).to(dev))
    torch.cuda.synchronize()
    t = ref.process(ref.params(**kw), p.left, p.right)
    check(e, t, oL.cpu().numpy(), oR.cpu().numpy())
    assert e.stats()["dense_evals"] == t.dense_evals


@pytest.mark.parametrize("kw", [{}, CENSUS], ids=["gradient", "census_median"])
def test_fused_match_in_mixed_batches(kw):
    """One call with both thread counts per row, and rows too wide for either."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1802_07210_amd as E
    kw = dict(disp_max=23, **kw)
    ps = [pair(w, h, 24) for w, h in [(640, 30), (641, 27), (65, 33), (705, 30), (3905, 31),
                                      (1537, 28), (640, 31), (2112, 26)]]
    dev = torch.device("cuda:0")
    e = E.Elas(**kw)
    items = []
    for p in ps:
        out = [torch.empty(p.left.shape, dtype=torch.int16, device=dev) for _ in range(2)]
        items.append((torch.from_numpy(p.left).to(dev), torch.from_numpy(p.right).to(dev), *out))
    e.process_batch(items)
    torch.cuda.synchronize()
    for p, (_, _, oL, oR) in zip(ps, items):
        t = ref.process(ref.params(**kw), p.left, p.right)
        assert np.array_equal(oL.cpu().numpy(), t.outL) and np.array_equal(oR.cpu().numpy(), t.outR)
