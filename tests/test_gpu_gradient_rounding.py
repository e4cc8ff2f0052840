"""The image gradient's fixed-point taps of levels of fronto planes round to
nearest: where one pixel's large gradient sets a coarse scale for its workgroup,
the others' small taps gather no bias."""
import numpy as np
import pytest

import scenegen
from scenegen import Level, Settings

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("window,n_src", [(5, 1), (7, 2), (9, 3)])
def test_taps_on_a_coarse_scale_have_no_bias(window, n_src):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1809_06132_amd.sweep import PlaneSweep, frame_to_device
    # one tile of 16 output rows and every lane: the large gradient's scale is
    # every workgroup's
    W, H, planes = 64, 16 + window - 1, 16
    fr = scenegen.random_small_frame(w=W, h=H, n_src=n_src, seed=40 + window, f=0.62 * W)
    lv = Level(n_fronto=16, near=1.0, far=15.0, window=window)
    ps = PlaneSweep(Settings(levels=[lv], best_k=min(2, n_src), mode="soft", temperature=0.1), W, H, n_src)
    ps.set_cameras(0, fr.ref_cam, fr.src_cams, fr.poses)
    out = ps.alloc_outputs()
    ps.run([frame_to_device(fr)], [out])
    usable = torch.isfinite(out["soft_invdepth"]).cpu().numpy()
    ys, xs = np.nonzero(usable)
    small = np.zeros((H, W), np.float32)
    small[usable] = np.random.default_rng(window).normal(size=usable.sum()).astype(np.float32)
    big = np.zeros((H, W), np.float32)
    big[ys[-1], xs[-1]] = 1.0   # the last usable pixel: its windows reach few others

    def grads(g):
        gs, _ = ps.soft_backward(torch.from_numpy(g).cuda(), [s.shape for s in fr.srcs])
        return np.stack([t.cpu().numpy() for t in gs]).astype(np.float64)

    # the small gradients alone have a fine scale; beside the large one their
    # texels are some thousand units
    eps = np.float32(2.0 ** -18)
    only_small, only_big, both = grads(eps * small), grads(big), grads(big + eps * small)
    ps.close()
    clean = (only_big == 0.0) & (only_small != 0.0)   # texels that only small taps reach
    want, got = only_small[clean], both[clean]
    assert clean.sum() > 200
    # the unit of the coarse sums: the largest power of two that divides them all
    unit = 2.0 ** 20
    while not np.array_equal(got / unit, np.rint(got / unit)):
        unit /= 2.0
    err = got - want
    taps = 4.0 * n_src * W * H * planes   # at most
    bias = float((err * np.sign(want)).sum()) / unit
    print(f"unit 2^{np.log2(unit):.0f}, typical texel {np.median(np.abs(want)) / unit:.0f} units, bias {bias:.1f} units "
          f"of {taps:.0f} taps, largest error {np.abs(err).max() / unit:.1f} units")
    assert np.median(np.abs(want)) / unit > 64 and np.abs(want).max() / unit < 2 ** 24
    # a tap rounded to nearest is off by a uniform half unit, of variance 1/12
    assert abs(bias) <= 6.0 * np.sqrt(taps / 12.0)
