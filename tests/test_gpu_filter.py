"""GPU depth-map filtering against the oracle's filter, on the same input
maps (the GPU sweep's own output, so both sides filter identical values)."""
import numpy as np
import pytest

import oracle
import scenegen

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _near_ratio(m, ratio):
    """Pixels whose cost2 / cost1 sits on the ratio threshold (to FP32
    rounding); invalid pixels (costs +inf) are not near it."""
    c1, c2 = m["cost1"].astype(np.float64), m["cost2"].astype(np.float64)
    fin = np.isfinite(c1) & np.isfinite(c2)
    near = np.zeros(c1.shape, bool)
    near[fin] = np.abs(c2[fin] - ratio * c1[fin]) <= 1e-6 * np.abs(c2[fin])
    return near


@pytest.mark.parametrize("window,ratio", [(5, 1.05), (3, 1.2), (7, 1.0)])
def test_filter_matches_oracle(window, ratio):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1809_06132_amd.sweep import PlaneSweep, frame_to_device
    wl = scenegen.workload("C1")
    fr, st = wl.frames[0], wl.settings
    ps = PlaneSweep(st, 320, 256, 1)
    ps.set_cameras(0, fr.ref_cam, fr.src_cams, fr.poses)
    out = ps.alloc_outputs()
    ps.run([frame_to_device(fr)], [out])
    d, c = ps.filter(out["merged"], ratio_min=ratio, window=window)
    torch.cuda.synchronize()
    m = {k: v.cpu().numpy() for k, v in out["merged"].items()}
    gd, gc = d.cpu().numpy(), c.cpu().numpy()
    ps.close()
    od, oc = oracle.depth_filter(fr.ref_cam, st.ground_n, m["depth"].astype(np.float64),
                                 m["cost1"].astype(np.float64), m["cost2"].astype(np.float64),
                                 ratio_min=ratio, window=window)
    # decisions can differ only where an FP32 comparison sits on its threshold
    near = _near_ratio(m, ratio)
    diff = (gc != oc) & ~near
    print("codes", np.bincount(gc.ravel(), minlength=256)[[0, 1, 2, 3, 255]], "mismatch", diff.sum())
    assert diff.sum() == 0
    keep = (gc == 0) & (oc == 0)
    assert np.array_equal(gd[keep], od[keep].astype(np.float32))
    assert np.all(np.isnan(gd[gc != 0]))


def test_mask_boxes_after_filter():
    """Detected boxes (some partly outside the image, overlapping, empty, and
    more than one launch holds) masked out of the filtered map, against the
    oracle's filter and mask."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1809_06132_amd.sweep import PlaneSweep, frame_to_device
    wl = scenegen.workload("C1")
    fr, st = wl.frames[0], wl.settings
    ps = PlaneSweep(st, 320, 256, 1)
    ps.set_cameras(0, fr.ref_cam, fr.src_cams, fr.poses)
    out = ps.alloc_outputs()
    ps.run([frame_to_device(fr)], [out])
    d, c = ps.filter(out["merged"])
    rng = np.random.default_rng(5)
    boxes = [(-20, -10, 40, 30), (300, 200, 400, 300), (100, 100, 100, 140), (50, 60, 120, 90), (70, 70, 130, 160)]
    boxes += [tuple(int(v) for v in (x, y, x + rng.integers(1, 30), y + rng.integers(1, 30)))
              for x, y in zip(rng.integers(-10, 320, 80), rng.integers(-10, 256, 80))]
    ps.mask_boxes(d, boxes, code=c)
    torch.cuda.synchronize()
    gd, gc = d.cpu().numpy(), c.cpu().numpy()
    m = {k: v.cpu().numpy() for k, v in out["merged"].items()}
    ps.close()
    od, oc = oracle.depth_filter(fr.ref_cam, st.ground_n, m["depth"].astype(np.float64),
                                 m["cost1"].astype(np.float64), m["cost2"].astype(np.float64))
    od, oc = oracle.mask_boxes(od, boxes, oc)
    near = _near_ratio(m, 1.05)
    assert ((gc != oc) & ~near).sum() == 0
    assert np.all(gc[oc == 4] == 4)
    keep = (gc == 0) & (oc == 0)
    assert np.array_equal(gd[keep], od[keep].astype(np.float32))
    assert np.all(np.isnan(gd[gc != 0]))

def test_filter_c2_full_map():
    """The filter on the full C2 map (1024x768, three sources, both plane
    families) against the oracle's filter of the same maps."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1809_06132_amd.sweep import PlaneSweep, frame_to_device
    wl = scenegen.workload("C2")
    fr, st = wl.frames[0], wl.settings
    ps = PlaneSweep(st, 1024, 768, 3)
    ps.set_cameras(0, fr.ref_cam, fr.src_cams, fr.poses)
    out = ps.alloc_outputs()
    ps.run([frame_to_device(fr)], [out])
    d, c = ps.filter(out["merged"])
    torch.cuda.synchronize()
    m = {k: v.cpu().numpy() for k, v in out["merged"].items()}
    gd, gc = d.cpu().numpy(), c.cpu().numpy()
    ps.close()
    od, oc = oracle.depth_filter(fr.ref_cam, st.ground_n, m["depth"].astype(np.float64),
                                 m["cost1"].astype(np.float64), m["cost2"].astype(np.float64))
    near = _near_ratio(m, 1.05)
    diff = (gc != oc) & ~near
    counts = np.bincount(gc.ravel(), minlength=256)[[0, 1, 2, 3, 255]]
    print("codes", counts, "mismatch", diff.sum())
    assert diff.sum() == 0
    assert counts[0] > 0.1 * gc.size and counts[1] > 0 and counts[3] > 0   # every filter acts
    keep = (gc == 0) & (oc == 0)
    assert np.array_equal(gd[keep], od[keep].astype(np.float32))
    assert np.all(np.isnan(gd[gc != 0]))


@pytest.mark.parametrize("window,w,h", [(3, 64, 16), (5, 65, 17), (7, 63, 15), (9, 130, 33), (11, 20, 12), (13, 200, 50),
                                        (15, 129, 70), (5, 8, 8)])
def test_filter_tile_edges_match_oracle(window, w, h):
    """Map sizes at and beside the filter's 64 x 16 tiles, smaller than its
    window, every window side; maps with holes, outliers and infinite values,
    and a pitch wider than the map."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1809_06132_amd import psweep as P
    from paper_1809_06132_amd.sweep import PlaneSweep
    rng = np.random.default_rng(100 * window + w)
    cam = scenegen.Camera(xi=0.9, fx=0.6 * w, fy=0.6 * w, cx=w / 2.0, cy=h / 2.0, width=w, height=h)
    st = scenegen.Settings(levels=[scenegen.Level(n_fronto=4, near=1.0, far=9.0, window=3)], best_k=1)
    ps = PlaneSweep(st, w, h, 1)
    ps.set_cameras(0, cam, [cam], [scenegen.Pose(R=np.eye(3), t=np.array([-0.3, 0.0, 0.0]))])
    pitch = w + 5
    d = (3.0 + 0.8 * rng.uniform(size=(h, pitch))).astype(np.float32)
    d[rng.uniform(size=d.shape) < 0.2] = 9.0
    d[rng.uniform(size=d.shape) < 0.1] = np.nan
    d[rng.uniform(size=d.shape) < 0.02] = np.inf
    c1 = (0.25 * rng.uniform(size=d.shape) ** 2).astype(np.float32)
    c2 = (c1 + 0.2 * rng.uniform(size=d.shape)).astype(np.float32)
    c1[np.isnan(d)] = np.inf
    c2[rng.uniform(size=d.shape) < 0.05] = np.inf
    t = [torch.from_numpy(a).cuda() for a in (d, c1, c2)]
    out = torch.full((h, pitch), 7.0, device="cuda")
    code = torch.full((h, pitch), 7, dtype=torch.uint8, device="cuda")
    m = P.psweep_maps(depth=t[0].data_ptr(), cost1=t[1].data_ptr(), cost2=t[2].data_ptr(), pitch=pitch)
    P.psweep_filter(ps.ctx, 0, m, P.psweep_filter_params(0.05, 0.3, 1.05, 0.5, 0.3, window), out.data_ptr(),
                    code.data_ptr(), pitch, int(torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    gd, gc = out.cpu().numpy(), code.cpu().numpy()
    ps.close()
    assert (gd[:, w:] == 7.0).all() and (gc[:, w:] == 7).all()
    d, c1, c2, gd, gc = d[:, :w], c1[:, :w], c2[:, :w], gd[:, :w], gc[:, :w]
    od, oc = oracle.depth_filter(cam, st.ground_n, d.astype(np.float64), c1.astype(np.float64), c2.astype(np.float64),
                                 window=window)
    near = _near_ratio({"cost1": c1, "cost2": c2}, 1.05)
    # a neighbour whose difference from the centre sits on gamma counts either way
    pad = np.pad(d.astype(np.float64), window // 2, constant_values=np.nan)
    tie = np.zeros(d.shape, bool)
    for j in range(window):
        for i in range(window):
            with np.errstate(invalid="ignore"):
                tie |= np.abs(np.abs(pad[j:j + h, i:i + w] - d) - 0.5) < 1e-6
    # and so may every pixel whose window holds a near-threshold ratio
    grow = np.pad(near, window // 2)
    near_win = np.zeros(d.shape, bool)
    for j in range(window):
        for i in range(window):
            near_win |= grow[j:j + h, i:i + w]
    assert ((gc != oc) & ~tie & ~near_win).sum() == 0
    keep = (gc == 0) & (oc == 0)
    assert np.array_equal(gd[keep], od[keep].astype(np.float32)) and np.all(np.isnan(gd[gc != 0]))
