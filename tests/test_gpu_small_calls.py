"""Parity with the oracle at the edges of the small-call paths: radix passes
without count launches (from about 2,000 points, up to eight frames and 2,048
filter chunks), chunk sizes of one, two and three tiles and of half a tile,
one to four passes, and frames over the cap of 16 and 17 steps of its flag
pass.  Structure bit for bit."""
import numpy as np
import pytest

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


@pytest.mark.parametrize("sizes,dims,cap", [
    ([2047], (256, 256, 16), 5000), ([2048], (256, 256, 16), 5000), ([2049], (2048, 2048, 64), 1000),
    ([16384], (512, 512, 32), 20000), ([16385], (512, 512, 32), 20000),
    ([131072], (128, 128, 8), 20000), ([131073], (512, 512, 32), 100000),
    ([300001], (256, 256, 16), 150000), ([300001], (16, 8, 4), 300000),
    ([30000, 0, 1, 20000, 4097, 2048, 0, 9999], (512, 512, 32), 15000),
    ([30000, 0, 1, 20000, 4097, 2048, 0, 9999, 5000], (512, 512, 32), 15000),
    ([100000, 20000, 5000], (2048, 2048, 64), 60000),
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v[0]) + f"of{len(v)}" if isinstance(v, list) else None)
def test_fold_edges(gpu_lib, sizes, dims, cap):
    case = _uniform(sizes, dims, cap)
    vz, exp = check(gpu_lib, case, label=f"{sizes} {dims}")
    vz.run()  # meets the first call's counts in its workspace
    assert_same_voxels(vz.result(), exp, feat_atol=FEAT_TOL, label="second call")
    assert vz.fault() == 0 and vz.header()["kept"] == sum(sizes)


@pytest.mark.parametrize("n", [524_288, 524_289])
def test_cap_steps_edge(gpu_lib, n):
    vz, exp = check(gpu_lib, _uniform([n, 70_000], (256, 256, 16), 150_000), label=f"cap {n}")
    assert vz.header()["capped_voxels"] > 150_000 and int(exp["voxel_offsets"][1]) == 150_000
