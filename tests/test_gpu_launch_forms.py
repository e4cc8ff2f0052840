"""The forms a winner-take-all run is launched in give the same maps, bit for
bit: the item queues of a grid config (one launch for every level, or for many
plane chunks) against a launch per job (what a timed run uses), and
psweep_run_noalloc with room for many plane chunks, few, and none, against
psweep_run in one pass."""
import dataclasses

import numpy as np
import pytest

import scenegen
from scenegen import Level, Settings
from tests.parity import to_np

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1809_06132_amd.sweep import PlaneSweep, frame_to_device
    return PlaneSweep, frame_to_device


def _frame(w, h, n_src, seed):
    fr = scenegen._street_frame(w, h, 0.3516 * w, 7100 + seed, 8100 + seed, ss=1, extra_right=True)
    return dataclasses.replace(fr, srcs=fr.srcs[:n_src], src_cams=fr.src_cams[:n_src], poses=fr.poses[:n_src])


def _one(nf, ng, win):
    return [Level(n_fronto=nf, near=0.5, far=30.0, n_ground=ng, window=win)]


def _two(w, h, nf, ng):
    return [Level(n_fronto=nf, near=0.5, far=30.0, n_ground=ng, window=7, downsample=2),
            Level(n_fronto=nf, near=5.0, far=60.0, n_ground=ng, window=9,
                  crop=((w - w // 2) // 2, (h - h // 2) // 2, w // 2, h // 2))]


def _marked(out):
    for t in out["merged"].values():
        t.fill_(7)
    return out


# sizes: one level whose items are more than the chip holds at once (the
# queues), with one output row of tiles, with a last tile column of one pixel,
# two levels of odd size, a level too small for a tile
@pytest.mark.parametrize("w,h,n_src,storage,levels", [
    (513, 301, 1, "f32", _one(40, 12, 9)), (640, 25, 2, "f32", _one(64, 0, 9)), (467, 400, 4, "f32", _one(70, 21, 7)),
    (401, 303, 3, "f32", _two(401, 303, 9, 5)), (333, 221, 4, "f16", _two(333, 221, 24, 0)),
    (260, 222, 2, "bf16", _two(260, 222, 13, 8)), (64, 40, 2, "f32", _two(64, 40, 6, 2)),
])
def test_queues_match_a_launch_per_job(w, h, n_src, storage, levels):
    PlaneSweep, frame_to_device = _gpu()
    fr = _frame(w, h, n_src, w % 7)
    ps = PlaneSweep(Settings(levels=levels, best_k=min(2, n_src)), w, h, n_src, storage=storage)
    ps.set_cameras(0, fr.ref_cam, fr.src_cams, fr.poses)
    d = frame_to_device(fr)
    got = {}
    for timed in (False, True, False):
        ps.set_timing(timed)
        for chunks in (0, 1, 5):
            for l in range(len(levels)):
                ps.set_chunks(l, chunks)
            out = _marked(ps.alloc_outputs())
            ps.run([d], [out])
            torch.cuda.synchronize()
            got[timed, chunks] = to_np(out["merged"])
    ps.close()
    want = got[True, 1]
    for k, m in got.items():
        for name in want:
            assert np.array_equal(want[name], m[name], equal_nan=True), (k, name)


# scratch beside the images for eight plane chunks (small), six, two and none;
# two levels; two frames
@pytest.mark.parametrize("w,h,n_src,levels,frames", [
    (200, 150, 2, _one(24, 10, 7), 1), (640, 480, 3, _one(30, 12, 9), 1), (1024, 768, 3, _one(10, 6, 9), 1),
    (1280, 832, 4, _one(8, 0, 9), 1), (512, 384, 3, _two(512, 384, 12, 6), 1), (301, 203, 2, _two(301, 203, 8, 0), 2),
])
def test_noalloc_matches_one_pass_at_its_scratch_limits(w, h, n_src, levels, frames):
    PlaneSweep, frame_to_device = _gpu()
    ps = PlaneSweep(Settings(levels=levels, best_k=2), w, h, n_src, max_frames=frames, max_camera_sets=frames)
    dev = []
    for f in range(frames):
        fr = _frame(w, h, n_src, f)
        ps.set_cameras(f, fr.ref_cam, fr.src_cams, fr.poses)
        dev.append(dict(frame_to_device(fr), camera_set=f))
    for l in range(len(levels)):
        ps.set_chunks(l, 1)
    want = [ps.alloc_outputs(camera_set=f) for f in range(frames)]
    ps.run(dev, want)
    for chunks in (0, 8):
        for l in range(len(levels)):
            ps.set_chunks(l, chunks)
        got = [_marked(ps.alloc_outputs(camera_set=f)) for f in range(frames)]
        ps.run_noalloc(dev, got)
        torch.cuda.synchronize()
        for a, b in zip(want, got):
            a, b = to_np(a["merged"]), to_np(b["merged"])
            assert (a["index"] >= 0).any()
            for name in a:
                assert np.array_equal(a[name], b[name], equal_nan=True), (chunks, name)
    ps.close()
