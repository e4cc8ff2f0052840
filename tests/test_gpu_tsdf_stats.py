"""Allocated blocks counted by one workgroup and by several (every block of one
integration has been seen, so the extracted counts say how many there are), and
the copy of boxes with rows of every length."""
import numpy as np
import pytest

import scenegen

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("blocks", [(5, 3, 9), (32, 32, 32), (33, 32, 32), (45, 41, 37)])
def test_stats_count_every_block(blocks):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1809_06132_amd.tsdf import TsdfMap
    seq = scenegen.depth_sequence(n_frames=1, w=160, h=120, seed=1011)
    tm = TsdfMap(voxel=0.1, mu=0.3, blocks=blocks, min_obs=1, max_width=160, max_height=120)
    tm.integrate(seq.cam, seq.poses[0], (0.0, 0.5, 4.0), torch.from_numpy(seq.depths[0]).cuda())
    allocated, visible = tm.stats()
    again = tm.stats()   # a call leaves nothing behind
    seen = int((tm.extract()["count"] > 0).sum())
    tm.close()
    assert allocated == seen > 0 and 0 < visible <= allocated and again == (allocated, visible)


@pytest.mark.parametrize("nx", [1, 2, 3, 5, 15, 16, 17, 31, 32, 33, 70])
def test_extraction_of_rows_of_any_length(nx):
    """The box's copy at row lengths around the number of half blocks that a
    wave holds, against a longer box with the same first block: the same sums
    there, bit for bit."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1809_06132_amd.tsdf import TsdfMap
    seq = scenegen.depth_sequence(n_frames=1, w=160, h=120, seed=1011)
    got = []
    for n in (nx, 72):
        tm = TsdfMap(voxel=0.1, mu=0.3, blocks=(n, 3, 9), min_obs=1, max_width=160, max_height=120)
        tm.integrate(seq.cam, seq.poses[0], (0.8 * (n // 2 - 1 + 0.5), 0.5, 4.0), torch.from_numpy(seq.depths[0]).cuda())
        e = tm.extract()
        got.append({k: t.cpu().numpy() if torch.is_tensor(t) else t for k, t in e.items()})
        tm.close()
    a, b = got
    assert np.array_equal(a["first_block"], b["first_block"]) and a["first_block"][0] == -1
    assert np.isfinite(a["tsdf"]).any() and (a["count"] > 0).any()
    for k, unit in (("tsdf", 8), ("weight", 8), ("count", 1)):
        assert np.array_equal(a[k], b[k][:, :, :unit * nx], equal_nan=True), k
