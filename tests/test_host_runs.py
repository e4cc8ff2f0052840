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


def test_tiles_without_a_grid_kernel_stay_refused(tmp_path):
    """A grid config with a tile shape that no grid kernel has is refused,
    whatever the persistent kernels are built for and however the run would be
    launched; a persistent config still takes the shapes it has."""
    out = host_run(tmp_path, """
        two = [(24, 0.5, 10, 7, 2, (0, 0, 0, 0)), (24, 0.5, 10, 9, 1, (128, 96, 256, 192))]
        one = [(60, 0.5, 20, 9, 1, (0, 0, 0, 0))]
        refused = 0
        for levels in (two, one):
            for store in (0, 1, 2):
                for S in (1, 2, 3, 4):
                    for tile in ((4, 4), (8, 4), (4, 8), (2, 8), (16, 4), (8, 2)):
                        got = {}
                        for launch, timed in ((0, True), (0, False), (1, False)):
                            r = Run(config(512, 384, S, levels, storage=store, launch=launch), 1 << 32)
                            for l in range(len(levels)):
                                P.psweep_set_tile(r.ctx, l, *tile)
                            P.psweep_set_timing(r.ctx, timed)
                            try:
                                r()
                                got[launch, timed] = 0
                            except P.PsweepError as e:
                                got[launch, timed] = e.status
                            P.psweep_destroy(r.ctx)
                        # a timed run is a launch per job: the grid kernels decide
                        assert got[0, False] == got[0, True], (len(levels), store, S, tile, got)
                        assert set(got.values()) <= {0, P.EUNSUPPORTED}
                        refused += got[0, False] != 0
                        if tile == (4, 8) and store == 2 and S >= 3:
                            assert got[0, False] == P.EUNSUPPORTED and got[1, False] == 0
        assert refused
        print("ok")
    """)
    assert "ok" in out
