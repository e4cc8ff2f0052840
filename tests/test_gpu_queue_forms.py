"""Item queues against a launch per job, with the form certain: a persistent
config always takes the queues, a timed grid config never does (the CPU tests of
the host side hold an untimed grid config's choice).  Every pass's maps are
compared, bit for bit."""
import dataclasses

import numpy as np
import pytest

import scenegen
from scenegen import Level, Settings
from tests.parity import to_np

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _frame(w, h, n_src, seed):
    fr = scenegen._street_frame(w, h, 0.3516 * w, 7300 + seed, 8300 + seed, ss=1, extra_right=True)
    return dataclasses.replace(fr, srcs=fr.srcs[:n_src], src_cams=fr.src_cams[:n_src], poses=fr.poses[:n_src])


def _one(nf, ng, win):
    return [Level(n_fronto=nf, near=0.5, far=30.0, n_ground=ng, window=win)]


def _two(w, h, nf, ng):
    return [Level(n_fronto=nf, near=0.5, far=30.0, n_ground=ng, window=7, downsample=2),
            Level(n_fronto=nf, near=5.0, far=60.0, n_ground=ng, window=9, crop=(w // 4, h // 4, w // 2, h // 2))]


# one row of tiles; one tile in one item, and in two (fewer than the queues);
# more items than the chip holds; two levels, one of them without a tile; frames
@pytest.mark.parametrize("w,h,n_src,storage,levels,frames", [
    (640, 24, 2, "f32", _one(64, 0, 9), 1), (60, 22, 1, "f32", _one(3, 0, 7), 1), (60, 22, 1, "f16", _one(8, 0, 7), 1),
    (513, 301, 1, "f32", _one(40, 12, 9), 1), (401, 303, 3, "bf16", _two(401, 303, 9, 5), 1),
    (40, 28, 2, "f32", _two(40, 28, 6, 2), 1), (200, 150, 4, "f16", _two(200, 150, 8, 4), 3),
])
def test_persistent_config_matches_a_launch_per_job(w, h, n_src, storage, levels, frames):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1809_06132_amd.sweep import PlaneSweep, frame_to_device
    sets = [_frame(w, h, n_src, f) for f in range(frames)]
    dev = [dict(frame_to_device(fr), camera_set=f) for f, fr in enumerate(sets)]
    got = {}
    # (launch, timed) of every pass; the maps start from a mark each time
    for launch, passes in (("grid", (True, False, True, False)), ("persistent", (False, True, False))):
        ps = PlaneSweep(Settings(levels=levels, best_k=min(2, n_src)), w, h, n_src, max_frames=frames, max_camera_sets=frames,
                        storage=storage, launch=launch)
        for f, fr in enumerate(sets):
            ps.set_cameras(f, fr.ref_cam, fr.src_cams, fr.poses)
        for n, timed in enumerate(passes):
            ps.set_timing(timed)
            for chunks in (0, 1, 5):
                for l in range(len(levels)):
                    ps.set_chunks(l, chunks)
                outs = [ps.alloc_outputs(camera_set=f) for f in range(frames)]
                for o in outs:
                    for t in o["merged"].values():
                        t.fill_(7)
                ps.run(dev, outs)
                torch.cuda.synchronize()
                if timed:   # a launch per job with a tile, or the run's one
                    _, launches = ps.sweep_kernel_ms()
                    assert launches <= (frames * len(levels) if launch == "grid" else 1)
                got[launch, n, timed, chunks] = [to_np(o["merged"]) for o in outs]
        ps.close()
    want = got["grid", 0, True, 1]
    assert any((m["index"] >= 0).any() for m in want)
    for key, maps in got.items():
        for f, m in enumerate(maps):
            for name in m:
                assert np.array_equal(want[f][name], m[name], equal_nan=True), (key, f, name)


@pytest.mark.parametrize("w,h,n_src,nf,ng,window,launch", [
    (64, 48, 3, 8, 0, 9, "grid"), (64, 48, 3, 8, 0, 9, "persistent"), (97, 61, 4, 2, 0, 5, "grid"), (160, 120, 2, 4, 2, 11, "grid"),
    (150, 90, 1, 5, 3, 7, "persistent"), (320, 256, 3, 16, 0, 13, "grid"), (640, 480, 1, 4, 2, 9, "grid"),
])
def test_automatic_chunks_match_one_pass(w, h, n_src, nf, ng, window, launch):
    """The chunks that the library chooses, down to one plane each, against one
    pass over all planes: the same maps, bit for bit."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1809_06132_amd.sweep import PlaneSweep, frame_to_device
    fr = _frame(w, h, n_src, window)
    ps = PlaneSweep(Settings(levels=_one(nf, ng, window), best_k=min(2, n_src)), w, h, n_src, launch=launch)
    ps.set_cameras(0, fr.ref_cam, fr.src_cams, fr.poses)
    got = []
    for chunks in (1, 0):
        ps.set_chunks(0, chunks)
        out = ps.alloc_outputs()
        for t in out["merged"].values():
            t.fill_(7)
        ps.run([frame_to_device(fr)], [out])
        torch.cuda.synchronize()
        got.append(to_np(out["merged"]))
    ps.close()
    assert (got[0]["index"] >= 0).any()
    for name in got[0]:
        assert np.array_equal(got[0][name], got[1][name], equal_nan=True), name
