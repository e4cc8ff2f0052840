"""What the host side gives the GPU, checked on the CPU (tests/fake_hip.py)."""
from tests.fake_hip import host_run


def test_noalloc_contexts_taking_turns(tmp_path):
    """psweep_run_noalloc from two contexts in turn: every run finds its own
    tables and plane setup in the scratch that they share, also where nothing
    of its own changed since its last call."""
    out = host_run(tmp_path, """
        a = Run(config(200, 150, 2, [(24, 0.5, 10, 7, 1, (0, 0, 0, 0))]), 1 << 32, t=0.1, workspace=False)
        b = Run(config(640, 480, 3, [(30, 0.7, 12, 9, 1, (0, 0, 0, 0))]), 1 << 33, t=0.3, workspace=False)
        c = Run(config(200, 150, 2, [(24, 0.9, 10, 7, 1, (0, 0, 0, 0))]), 1 << 34, t=0.5, workspace=False)
        for who in (a, b, a, a, c, a, b, c, c):
            log = who(P.psweep_run_noalloc)
            got = sweeps(log)
            assert len(got) == 1, log
            g, cfg = got[0], who.cfg
            want = dict(w=cfg.max_width, h=cfg.max_height, src=cfg.max_sources, window=cfg.level[0].window, inside=1,
                        index=who.outs[0].merged.index)
            assert all(g[k] == v for k, v in want.items()), (g, want)
            plane0 = cfg.level[0].near_m + 100 * (0.1 if who is a else 0.3 if who is b else 0.5)
            assert abs(g["plane0"] - plane0) < 1e-3, (g, plane0)
        # a context that has the scratch to itself uploads nothing again
        assert "upload" not in c(P.psweep_run_noalloc)
        # and one that is destroyed leaves nothing behind for a later one
        P.psweep_destroy(c.ctx)
        d = Run(c.cfg, 1 << 34, t=0.7, workspace=False)
        assert abs(sweeps(d(P.psweep_run_noalloc))[0]["plane0"] - 70.9) < 1e-3
        print("ok")
    """)
    assert "ok" in out
