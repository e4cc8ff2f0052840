"""psweep_run_noalloc from contexts that take turns on one GPU: its static
scratch holds one run's tables, so a context that comes back, with nothing of
its own changed, has to set them up again."""
import threading

import numpy as np
import pytest

import scenegen
from scenegen import Level, Settings
from tests.parity import to_np

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _context(w, h, n_src, nf, ng, win, seed):
    from paper_1809_06132_amd.sweep import PlaneSweep, frame_to_device
    fr = scenegen.random_small_frame(w=w, h=h, n_src=n_src, seed=seed, f=0.5 * w)
    st = Settings(levels=[Level(n_fronto=nf, near=0.5, far=30.0, n_ground=ng, window=win)], best_k=min(2, n_src))
    ps = PlaneSweep(st, w, h, n_src)
    ps.set_cameras(0, fr.ref_cam, fr.src_cams, fr.poses)
    frame, want, got = frame_to_device(fr), ps.alloc_outputs(), ps.alloc_outputs()
    ps.run([frame], [want])
    torch.cuda.synchronize()
    return ps, frame, to_np(want["merged"]), got


def _check(got, want, what):
    torch.cuda.synchronize()
    g = to_np(got["merged"])
    assert (want["index"] >= 0).any()
    for k in want:
        assert np.array_equal(want[k], g[k], equal_nan=True), (what, k)


# other sizes and source counts, one and several plane chunks, a launch per job
# and item queues
SHAPES = [(200, 150, 2, 24, 10, 7, 91), (640, 480, 3, 30, 12, 9, 92), (97, 64, 1, 8, 0, 5, 93)]


def test_contexts_taking_turns():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = [_context(*s) for s in SHAPES]
    for turn, i in enumerate((0, 1, 0, 0, 2, 1, 2, 0)):
        ps, frame, want, got = ctx[i]
        others = [(j, {k: t.clone() for k, t in c[3]["merged"].items()}) for j, c in enumerate(ctx) if j != i]
        for t in got["merged"].values():
            t.fill_(7)
        ps.run_noalloc([frame], [got])
        _check(got, want, (turn, i))
        for j, before in others:   # and nobody else's maps are touched
            for k, t in before.items():
                assert torch.equal(t.nan_to_num(), ctx[j][3]["merged"][k].nan_to_num()), (turn, i, j, k)
    for c in ctx:
        c[0].close()


def test_threads_taking_turns_on_one_stream():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = [_context(*s) for s in SHAPES[:2]]
    errors = []

    def serve(c):
        try:
            for _ in range(20):
                c[0].run_noalloc([c[1]], [c[3]])
        except Exception as e:   # shown by the main thread
            errors.append(e)

    threads = [threading.Thread(target=serve, args=(c,)) for c in ctx]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for i, c in enumerate(ctx):
        _check(c[3], c[2], i)
        c[0].close()
