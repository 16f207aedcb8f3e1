"""Rows too wide for matching and check in one kernel (more than 2112 columns,
census 3840): the separate kernels, at every dense tile height, in single calls,
batches, and batches whose descriptors go past the last-level cache (192 MiB).
Raw and final maps must equal the oracle's."""
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
    cfg = synth.SceneConfig(w, h, D, 9, 0.05, 4.0, D - 5.0, 2.0, 0.10, patch=24, seed=seed)
    return synth.make_pair(cfg)


def on_gpu(p):
    dev = torch.device("cuda:0")
    L, R = torch.from_numpy(p.left).to(dev), torch.from_numpy(p.right).to(dev)
    oL = torch.full(L.shape, -7, dtype=torch.int16, device=dev)
    return L, R, oL, torch.full_like(oL, -7)


def same(get, out, t):
    assert np.array_equal(get("raw_left").reshape(t.rawL.shape), t.rawL)
    assert np.array_equal(get("raw_right").reshape(t.rawR.shape), t.rawR)
    assert np.array_equal(out[2].cpu().numpy(), t.outL)
    assert np.array_equal(out[3].cpu().numpy(), t.outR)


# heights that no tile height divides, one below a tile; the first column counts past the limits
@pytest.mark.parametrize("w,h,D,kw", [(2113, 37, 32, {}), (2369, 11, 256, {}), (2200, 50, 64, dict(full_search=1)),
                                      (3841, 27, 48, dict(descriptor=1))])
@pytest.mark.parametrize("rows", [1, 2, 4])
@pytest.mark.parametrize("batched", [False, True])
def test_dense_tiles_of_wide_rows(E, w, h, D, kw, rows, batched):
    p = pair(w, h, D, 5)
    t = ref.process(ref.params(disp_max=D - 1, **kw), p.left, p.right)
    assert (t.outL >= 0).any()
    e = E.Elas(disp_max=D - 1, **kw)
    e.set_tile_variants(w, h, 8, rows, 16)
    assert e.tuned_variants(w, h) == (8, rows, 16)
    items = [on_gpu(p) for _ in range(3 if batched else 1)]
    if batched:
        for _ in range(2):  # captured, then replayed
            e.process_batch(items)
        torch.cuda.synchronize()
        for i in range(3):
            same(lambda name: e.batch_intermediate(i, name), items[i], t)
    else:
        e.process(*items[0])
        torch.cuda.synchronize()
        assert e.stats()["dense_evals"] == t.dense_evals
        same(e.intermediate, items[0], t)


@pytest.mark.parametrize("rows", [1, 2, 4])
def test_dense_tiles_of_a_batch_past_the_cache(E, rows):
    w, h, D, n = 2117, 61, 48, 50
    assert 32 * w * h * n >= 192 << 20
    pairs = [pair(w, h, D, s) for s in range(3)]
    want = [ref.process(ref.params(disp_max=D - 1), p.left, p.right) for p in pairs]
    e = E.Elas(disp_max=D - 1)
    e.set_tile_variants(w, h, 8, rows, 16)
    items = [on_gpu(pairs[i % 3]) for i in range(n)]
    for _ in range(2):
        e.process_batch(items)
    torch.cuda.synchronize()
    for i in range(n):
        assert np.array_equal(items[i][2].cpu().numpy(), want[i % 3].outL)
        assert np.array_equal(items[i][3].cpu().numpy(), want[i % 3].outR)
    same(lambda name: e.batch_intermediate(n - 1, name), items[n - 1], want[(n - 1) % 3])


def test_a_size_tuned_for_both_descriptors(E):
    """At 2120 columns census rows are matched and checked in one kernel, gradient
    rows are not: one call with both, tuned together."""
    w, h, D = 2120, 40, 32
    p = pair(w, h, D, 8)
    census, plain = E.Elas(disp_max=D - 1, descriptor=1), E.Elas(disp_max=D - 1)
    for order in ((census, plain), (plain, census)):
        e = E.Elas(disp_max=D - 1)
        items = [on_gpu(p) + (q,) for q in order]
        for _ in range(2):
            e.process_batch(items)
        torch.cuda.synchronize()
        assert e.tuned_variants(w, h)[1] in (1, 2, 4)
        for i, q in enumerate(order):
            t = ref.process(ref.params(disp_max=D - 1, descriptor=int(q is census)), p.left, p.right)
            same(lambda name: e.batch_intermediate(i, name), items[i], t)
