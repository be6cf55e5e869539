"""Parity with the oracle at the edges of the small-call paths: radix passes
without count launches (up to eight frames and 2,048 filter chunks, where the
passes' count rows fit: 2,304 points for one frame of three passes, 393,216
for eight), on both sides of that line, with one to four passes, 64 and 128
chunks a frame, chunks of half a tile and of one, two and three tiles, empty
frames and frames of one point; which path ran is asserted.  And frames over
the cap of 16 and 17 steps of its flag pass (a large call).  Structure bit for
bit."""
import ctypes

import numpy as np
import pytest
import torch

from common import Case, assert_same_voxels, records
from test_gpu_parity import FEAT_TOL, check

pytestmark = pytest.mark.gpu


def _uniform(sizes, dims, cap, max_points=4, seed=3):
    """Frames of the given numbers of points, uniform over the grid, one ROI over all of it: every point is kept."""
    rng = np.random.default_rng(seed)
    B, N, voxel = len(sizes), int(sum(sizes)), (0.2, 0.2, 0.25)
    mn = (-0.1 * dims[0], -0.1 * dims[1], -2.0)
    cols = [mn[d] + (0.001 + 0.998 * rng.random(N)) * dims[d] * voxel[d] for d in range(3)]
    feat = np.ascontiguousarray(np.stack(cols + [rng.random(N)]).astype(np.float32))
    pose = np.array([1, 0, 0, 0, 0, 1, 0, 0, 0, 0, 1, 0], np.float32)
    grid = dict(range_min=list(mn), voxel_size=list(voxel), dims=list(dims), max_points=max_points, max_voxels=cap,
                num_sweeps=1, num_frames=B)
    return Case(feat=feat, sweep_ids=np.zeros(N, np.uint8), frame_offsets=np.concatenate([[0], np.cumsum(sizes)]),
                poses=np.tile(pose, (B, 1)).reshape(B, 1, 12), rois=records([[0.0, 0.0, 1.0, 0.0, 1e4, 1e4]] * B),
                roi_offsets=np.arange(B + 1, dtype=np.int32), budgets=np.ones(B, np.uint8), grid=grid)


def _launches(mb, vz):
    """Kernel launches of a call: the nodes of its captured graph (no count launches: filter, compaction, one scatter a
    pass, heads, finalisation, mean)."""
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        vz.run()
    n = ctypes.c_size_t(0)
    assert mb.load().hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    return n.value


# the last two: the call's launches (8 with three passes counted by the launch
# before, 11 with count launches, 12 with a segments launch too) and its pair
# chunks (in frames of up to 128 or 64 of them: rows for that many are there
# from 32,768 or 16,384 points per pass and frame on, fewer are for small frames)
@pytest.mark.parametrize("sizes,dims,cap,launches,chunks", [
    ([2047], (256, 256, 16), 5000, 8, 2),
    ([2048], (256, 256, 16), 5000, 11, 2),
    ([2303], (256, 256, 16), 5000, 11, 3),
    ([2304], (256, 256, 16), 5000, 8, 3),
    ([2049], (2048, 2048, 64), 1000, 13, 3),
    ([16384], (512, 512, 32), 20000, 8, 16),
    ([16385], (512, 512, 32), 20000, 8, 9),
    ([131072], (128, 128, 8), 20000, 7, 64),
    ([131073], (512, 512, 32), 100000, 8, 65),
    ([300001], (256, 256, 16), 150000, 8, 74),
    ([300001], (16, 8, 4), 300000, 6, 74),
    ([65535], (2048, 2048, 64), 70000, 13, 32),
    ([65536], (2048, 2048, 64), 70000, 9, 32),
    ([523264], (256, 256, 16), 150000, 8, 128),
    ([523265], (256, 256, 16), 150000, 12, 64),
    ([30000, 0, 1, 20000, 4097, 2048, 0, 9999], (512, 512, 32), 15000, 11, 43),
    ([30000, 0, 1, 20000, 4097, 2048, 0, 9999, 5000], (512, 512, 32), 15000, 11, 48),
    ([100000, 20000, 5000], (2048, 2048, 64), 60000, 13, 64),
    ([90000, 8304], (512, 512, 32), 50000, 8, 53),
    ([120000, 20000, 8000], (512, 512, 32), 60000, 8, 77),
    ([280000, 10000, 5000], (512, 512, 32), 200000, 8, 84),
    ([100000, 31072], (2048, 2048, 64), 60000, 9, 65),
    ([100000, 80000, 30000], (2048, 2048, 64), 90000, 9, 104),
    ([0, 393216, 0], (2048, 2048, 64), 200000, 9, 96),
    ([300000] + [13317] * 7, (512, 512, 32), 100000, 8, 147),
    ([300000, 0, 1, 20000, 4097, 2048, 0, 67074], (512, 512, 32), 60000, 8, 100),
    ([300000, 0, 1, 20000, 4097, 2048, 0, 67074, 5000], (512, 512, 32), 60000, 11, 105),
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v[0]) + f"of{len(v)}" if isinstance(v, list) else None)
def test_fold_edges(gpu_lib, sizes, dims, cap, launches, chunks):
    case = _uniform(sizes, dims, cap)
    vz, exp = check(gpu_lib, case, label=f"{sizes} {dims}")
    vz.run()  # meets the first call's counts in its workspace
    assert_same_voxels(vz.result(), exp, feat_atol=FEAT_TOL, label="second call")
    assert vz.fault() == 0 and vz.header()["kept"] == sum(sizes)
    assert vz.header()["pair_chunks"] == chunks and _launches(gpu_lib, vz) == launches


@pytest.mark.parametrize("n", [524_288, 524_289])
def test_cap_steps_edge(gpu_lib, n):
    vz, exp = check(gpu_lib, _uniform([n, 70_000], (256, 256, 16), 150_000), label=f"cap {n}")
    assert vz.header()["capped_voxels"] > 150_000 and int(exp["voxel_offsets"][1]) == 150_000
