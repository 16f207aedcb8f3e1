"""Past-only redundancy and down-sampling at the lattice sizes where their
kernels change form: the lattice staged in LDS (at most 76800 points) or
walked in global memory, the unrolled default distance and the general one,
and survivor counts over lattices that are no multiple of eight."""
import numpy as np
import pytest

import synth
from oracle import ref

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("w,h,step,dist", [(316, 261, 1, 5), (316, 261, 1, 7), (310, 259, 1, 5),
                                           (61, 47, 1, 5), (33, 19, 5, 5), (131, 90, 3, 6)])
def test_past_only_redundancy_sizes(w, h, step, dist):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1802_07210_amd as E
    p = synth.make_pair(synth.SceneConfig(w, h, 16, 4, 0.05, 2.0, 13.0, 2.0, 0.05, seed=w + dist))
    kw = dict(disp_max=15, candidate_stepsize=step, redundancy=1, redun_max_dist=dist,
              support_subsample=3)
    e = E.Elas(**kw)
    dev = torch.device("cuda:0")
    oL, oR = e.process(torch.from_numpy(p.left).to(dev), torch.from_numpy(p.right).to(dev))
    torch.cuda.synchronize()
    t = ref.process(ref.params(**kw), p.left, p.right)
    lh, lw = t.dcan_raw.shape
    assert (lw * lh > 76800) == (w == 316)
    for name, want in (("dcan_vert", t.dcan_vert), ("dcan_final", t.dcan_final)):
        assert np.array_equal(e.intermediate(name).reshape(lh, lw), want), name
    assert np.array_equal(e.intermediate("support_left").reshape(-1, 3), t.ptsL)
    assert np.array_equal(e.intermediate("support_right").reshape(-1, 3), t.ptsR)
    assert np.array_equal(oL.cpu().numpy(), t.outL) and np.array_equal(oR.cpu().numpy(), t.outR)
