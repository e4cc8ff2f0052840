"""Drives the host side of the built libpsweep.so on the CPU: tests/c/fake_hip.cpp
is loaded in place of the HIP runtime and logs every launch with what its
tables say.  `host_run(tmp_path, script)` runs `script` in a child process with
the names below and returns what it printed."""
import os
import subprocess
import sys
import textwrap

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

_PRELUDE = """
import ctypes
import re
import sys
# first in the global scope: the library's HIP calls find these
FAKE = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
FAKE.fake_hip_log.restype = ctypes.c_char_p
from paper_1809_06132_amd import psweep as P
ctypes.CDLL(P.LIB_PATH, mode=ctypes.RTLD_GLOBAL)

def config(w, h, n_src, levels, frames=1, **kw):
    # levels: (fronto planes, near, ground planes, window, downsample, crop)
    c = P.psweep_config()
    c.n_levels = len(levels)
    for l, (nf, near, ng, win, ds, crop) in enumerate(levels):
        L = c.level[l]
        L.n_fronto, L.near_m, L.far_m, L.n_ground, L.h_lo, L.h_hi = nf, near, 30.0, ng, -0.3, 0.3
        L.window, L.downsample = win, ds
        L.crop_x, L.crop_y, L.crop_w, L.crop_h = crop
    c.ground_n[:] = [0.0, 1.0, 0.0]
    c.ground_d, c.best_k, c.var_floor, c.temperature = 1.5, min(2, n_src), 1.0, 0.1
    c.max_width, c.max_height, c.max_sources, c.max_frames, c.max_camera_sets = w, h, n_src, frames, frames
    for k, v in kw.items():
        setattr(c, k, v)
    return c

class Run:
    # a context with cameras, and frames and maps that are addresses only:
    # nothing behind them is ever read
    def __init__(self, cfg, at, t=0.1, workspace=True):
        self.cfg, self.ctx = cfg, P.psweep_create(cfg)
        w, h, S = cfg.max_width, cfg.max_height, cfg.max_sources
        cam = P.psweep_camera(0.9, 0.5 * w, 0.5 * w, w / 2.0, h / 2.0, w, h)
        poses = [P.psweep_pose((P._d * 9)(1, 0, 0, 0, 1, 0, 0, 0, 1), (P._d * 3)(t * (s + 1), 0, 0)) for s in range(S)]
        self.frames, self.outs = [], []
        for f in range(cfg.max_frames):
            P.psweep_set_cameras(self.ctx, f, cam, [cam] * S, poses)
            fr = P.psweep_frame(ref=at, ref_pitch=w, camera_set=f)
            for s in range(S):
                fr.src[s], fr.src_pitch[s] = at + 4096 * (s + 1), w
            o = P.psweep_output()
            o.merged = P.psweep_maps(*[at + (1 << 20) * (m + 1) + 65536 * f for m in range(7)], 0)
            self.frames.append(fr)
            self.outs.append(o)
        if workspace:
            n = P.psweep_workspace_size(self.ctx)
            self.mem = ctypes.create_string_buffer(n + 256)
            P.psweep_set_workspace(self.ctx, (ctypes.addressof(self.mem) + 255) // 256 * 256, n)

    def __call__(self, call=P.psweep_run):
        FAKE.fake_hip_clear()
        call(self.ctx, self.frames, self.outs)
        return FAKE.fake_hip_log().decode().splitlines()

def sweeps(log):
    # the sweep launches' jobs as dicts
    out = []
    for l in log:
        if l.startswith(("grid", "queues")):
            d = dict(re.findall(r"(\\w+)=(\\S+)", l))
            out.append(dict({k: v if k == "tile" else float(v) for k, v in d.items()}, form=l.split()[0]))
    return out
"""


def host_run(tmp_path, script):
    from paper_1809_06132_amd import psweep
    if not os.path.exists(psweep.LIB_PATH):
        pytest.skip("libpsweep.so not built (run __graft_entry__.build())")
    fake = tmp_path / "libfake_hip.so"
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           os.path.join(ROOT, "tests", "c", "fake_hip.cpp"), "-o", str(fake), "-ldl"])
    env = dict(os.environ, PYTHONPATH=ROOT)
    r = subprocess.run([sys.executable, "-c", _PRELUDE + textwrap.dedent(script), str(fake)], capture_output=True,
                       text=True, env=env, cwd=str(tmp_path), timeout=300)
    assert r.returncode == 0, f"ended with {r.returncode}\n" + (r.stdout + r.stderr)[-6000:]
    return r.stdout
