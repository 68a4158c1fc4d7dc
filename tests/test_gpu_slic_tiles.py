"""GPU segmentation at the edges of its tiles (64 x 32 pixels per block, eight rows per thread, sums per block): labels,
segment counts and boundary table against the oracle's exact integer arithmetic, on rough pointmaps with holes and
low-confidence pixels so that members jump between cells."""
import numpy as np
import pytest
import torch

from oracle import depth as D

pytestmark = pytest.mark.gpu

ds3 = pytest.importorskip("paper_2605_30488_amd.api")


# one tile and a pixel less or more each way; a cell of one pixel; cells larger than a tile; several image shapes at once
@pytest.mark.parametrize("shapes,M", [([(32, 64)], 60), ([(31, 63)], 60), ([(33, 65)], 60), ([(8, 9)], 72),
                                      ([(100, 230)], 4), ([(65, 129), (33, 64), (7, 200)], 40)])
def test_labels_at_tile_edges(shapes, M):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(sum(h * w for h, w in shapes))
    xyz, conf = [], []
    for H, W in shapes:
        v, u = np.mgrid[0:H, 0:W]
        z = 5 + np.sin(u / 7.0) + np.cos(v / 5.0) + 0.05 * rng.normal(size=(H, W)) + 2.0 * (u > W // 2)
        x = np.stack([(u - W / 2) / W * z, (v - H / 2) / W * z, z], -1).astype(np.float32)
        x[rng.uniform(size=(H, W)) < 0.03] = 0.0
        xyz.append(x)
        conf.append(rng.uniform(1.3, 5, size=(H, W)).astype(np.float32))
    dev = torch.device("cuda:0")
    a = ds3.build_arena(xyz, conf, "f32", dev)
    p = ds3.default_depth_params()
    p.segments_per_kf, p.min_seg_px = M, 3
    plan = ds3.DepthPlan(ds3.Graph(a, [], torch.zeros(1, dtype=torch.int32, device=dev)), p)
    prob = D.DepthProblem(xyz, conf, [], [], params=D.DepthParams(segments_per_kf=M, min_seg_px=3))
    lab = plan.labels().cpu().numpy()
    for k, (H, W, off) in enumerate(a.images):
        assert np.array_equal(lab[off:off + H * W], prob.glabel(k)), k
    assert plan.info["segments"] == prob.n_seg
    assert plan.info["valid_segments"] == int(prob.seg_valid.sum())
    assert plan.info["boundary_slots"] == len(prob.pairs)
    plan.close()
