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


def test_launch_form_of_one_job(tmp_path):
    """A grid config's single job goes into the item queues only where its grid's
    items, in the chunks that it would have, are more than the chip holds (here
    256 CUs of four workgroups) and its tiles are long; several jobs always do.
    The chunks a caller sets, and those the static scratch has room for, count as
    they are."""
    out = host_run(tmp_path, """
        def form(w, h, S, planes, win=7, chunks=0, call=P.psweep_run, frames=1, ground=0, **kw):
            r = Run(config(w, h, S, [(planes, 0.5, ground, win, 1, (0, 0, 0, 0))], frames=frames, **kw), 1 << 32,
                    workspace=call is P.psweep_run)
            P.psweep_set_chunks(r.ctx, 0, chunks)
            got = sweeps(r(call))
            assert all(g["inside"] == 1 for g in got), got
            P.psweep_destroy(r.ctx)
            return got[0]["form"], got[0]["chunks"], got[0]["items"]

        # 320x256, window 7: 6 x 16 tiles
        assert form(320, 256, 1, 32) == ("grid", 7, 672)
        # 10 x 20 tiles: five chunks, not the eight that 32 planes allow
        assert form(586, 326, 1, 32) == ("grid", 5, 1000)
        assert form(586, 326, 1, 32, chunks=5) == ("grid", 5, 1000)
        assert form(640, 480, 3, 96, chunks=1)[:2] == ("grid", 1)
        assert form(640, 480, 3, 96)[0] == "queues"
        assert form(640, 480, 3, 96, frames=2, chunks=1)[0] == "queues"
        # more items than places, but short tiles, or tiles mostly of ground planes
        assert form(1024, 768, 1, 34, ground=55)[0] == "grid"
        assert form(1206, 919, 2, 34, 9, ground=55)[0] == "grid"
        assert form(586, 342, 2, 16, 9, ground=64)[0] == "grid"
        assert form(640, 480, 4, 30, ground=100)[0] == "grid"
        assert form(801, 601, 2, 128, storage=P.STORAGE_BF16)[0] == "queues"
        assert form(640, 480, 3, 64, 9, ground=30)[0] == "queues"
        # four sources in FP32: at window 9 whatever the tiles
        assert form(1206, 919, 4, 64, 9, ground=30)[0] == "queues"
        assert form(1206, 919, 4, 64, 7, ground=30)[0] == "grid"
        assert form(1206, 919, 4, 64, 9, ground=30, storage=P.STORAGE_F16)[0] == "grid"
        # a persistent config is never a grid
        assert form(320, 256, 1, 32, launch=1)[0] == "queues"
        # the static scratch with no room for chunks
        assert form(1024, 896, 4, 200, call=P.psweep_run_noalloc) == ("grid", 1, 1008)
        assert form(896, 608, 3, 200, 9, call=P.psweep_run_noalloc)[0] == "queues"
        print("ok")
    """)
    assert "ok" in out


def test_queues_hold_every_item_once(tmp_path):
    """Runs in the item queues: one row of tiles, fewer items than queues, a
    level too small for a tile, many frames; every job's items are all there."""
    out = host_run(tmp_path, """
        small = (16, 0.5, 0, 7, 1, (0, 0, 0, 0))
        for w, h, S, levels, frames, kw in (
                (640, 22, 2, [(64, 0.5, 0, 9, 1, (0, 0, 0, 0))], 1, dict(launch=1)),        # 12 x 1 tiles
                (60, 22, 1, [(8, 0.5, 0, 7, 1, (0, 0, 0, 0))], 1, dict(launch=1)),          # one tile, two chunks
                (60, 22, 1, [(3, 0.5, 0, 7, 1, (0, 0, 0, 0))], 1, dict(launch=1)),          # one item
                (40, 12, 2, [(8, 0.5, 0, 7, 2, (0, 0, 0, 0)), (8, 0.5, 0, 7, 1, (4, 0, 16, 12))], 1, {}),
                (320, 200, 2, [small], 16, {}), (1024, 544, 4, [(64, 0.5, 30, 7, 2, (0, 0, 0, 0)),
                                                               (64, 0.5, 30, 9, 1, (256, 128, 512, 272))], 1, {})):
            r = Run(config(w, h, S, levels, frames=frames, **kw), 1 << 32)
            got = sweeps(r())
            assert len(got) == frames * len(levels) and all(g["form"] == "queues" for g in got), got
            for g, lv in zip(got, levels * frames):
                hw = lv[3] // 2
                tiles = max(0, -(-(int(g["w"]) - 2 * hw) // (64 - 2 * hw))) * max(0, -(-(int(g["h"]) - 2 * hw) // 16))
                assert g["inside"] == 1 and g["items"] == tiles * g["chunks"], (g, tiles)
        print("ok")
    """)
    assert "ok" in out


def test_tsdf_stats_of_large_maps_take_many_workgroups(tmp_path):
    """The allocated blocks of a map are counted by workgroups in proportion to
    its slots, after one launch that clears their sum."""
    out = host_run(tmp_path, """
        for blocks, launches in (((75, 4, 75), [1]), ((32, 32, 32), [1]), ((33, 32, 32), [1, 9]), ((256, 256, 256), [1, 256])):
            c = P.psweep_tsdf_config(0.1, 0.3, (P._i32 * 3)(*blocks), 100.0, 1, 160, 120)
            ts = P.psweep_tsdf_create(c)
            # an address only: the launches are not played
            P.psweep_tsdf_set_workspace(ts, 1 << 36, P.psweep_tsdf_workspace_size(ts))
            P.psweep_tsdf_reset(ts)
            cam = P.psweep_camera(0.9, 80.0, 80.0, 80.0, 60.0, 160, 120)
            pose = P.psweep_pose((P._d * 9)(1, 0, 0, 0, 1, 0, 0, 0, 1), (P._d * 3)(0, 0, 0))
            P.psweep_tsdf_integrate(ts, cam, pose, (0.0, 0.0, 0.0), 1 << 32, 0)
            FAKE.fake_hip_clear()
            P.psweep_tsdf_stats(ts, 1 << 33)
            got = [int(l.split("=")[1]) for l in FAKE.fake_hip_log().decode().splitlines()]
            assert got == launches, (blocks, got)
            P.psweep_tsdf_destroy(ts)
        print("ok")
    """)
    assert "ok" in out


def test_tsdf_extraction_fills_its_waves_in_narrow_boxes(tmp_path):
    """The copy of a box takes a lane per half a block's row: rows of few blocks
    share a wave, so that the workgroups go down with them."""
    out = host_run(tmp_path, """
        for blocks in ((1, 64, 64), (2, 64, 64), (3, 5, 7), (16, 8, 8), (17, 8, 8), (32, 8, 8), (75, 4, 75)):
            c = P.psweep_tsdf_config(0.1, 0.3, (P._i32 * 3)(*blocks), 100.0, 1, 160, 120)
            ts = P.psweep_tsdf_create(c)
            P.psweep_tsdf_set_workspace(ts, 1 << 36, P.psweep_tsdf_workspace_size(ts))
            P.psweep_tsdf_reset(ts)
            cam = P.psweep_camera(0.9, 80.0, 80.0, 80.0, 60.0, 160, 120)
            pose = P.psweep_pose((P._d * 9)(1, 0, 0, 0, 1, 0, 0, 0, 1), (P._d * 3)(0, 0, 0))
            P.psweep_tsdf_integrate(ts, cam, pose, (0.0, 0.0, 0.0), 1 << 32, 0)
            FAKE.fake_hip_clear()
            P.psweep_tsdf_extract(ts, 1 << 33, 1 << 34, 1 << 35)
            got = [int(l.split("=")[1]) for l in FAKE.fake_hip_log().decode().splitlines()]
            rows, per_wave = blocks[1] * blocks[2] * 64, max(1, 64 // (2 * blocks[0]))
            assert got == [-(-rows // (4 * per_wave))], (blocks, got)
            P.psweep_tsdf_destroy(ts)
        print("ok")
    """)
    assert "ok" in out


def test_plane_chunks_of_small_and_of_large_runs(tmp_path):
    """Automatic plane chunks: as short as a plane where the run leaves the chip
    empty, one or two a tile where its tiles alone fill it several times over."""
    out = host_run(tmp_path, """
        def auto(w, h, S, planes, win, **kw):
            r = Run(config(w, h, S, [(planes, 0.5, 0, win, 1, (0, 0, 0, 0))], **kw), 1 << 32)
            got = sweeps(r())
            P.psweep_destroy(r.ctx)
            assert got[0]["inside"] == 1
            return got[0]["form"], got[0]["chunks"]

        assert auto(64, 48, 3, 8, 9) == ("grid", 8)
        assert auto(64, 48, 3, 8, 9, launch=1) == ("queues", 8)
        assert auto(160, 120, 3, 6, 5) == ("grid", 6)
        assert auto(96, 64, 4, 2, 9) == ("grid", 2)
        assert auto(64, 48, 1, 3, 9) == ("grid", 1)         # three steps stay whole
        assert auto(640, 480, 3, 8, 9) == ("grid", 2)       # 360 tiles
        assert auto(1024, 768, 1, 16, 5) == ("grid", 1)     # 816 tiles, r 1.58
        assert auto(1280, 960, 1, 48, 5) == ("grid", 2)     # 1,320 tiles, r 2.2
        assert auto(1024, 768, 1, 48, 5) == ("grid", 4)     # r 2.7
        assert auto(2048, 1536, 1, 16, 5) == ("grid", 1)    # 3,360 tiles
        print("ok")
    """)
    assert "ok" in out
