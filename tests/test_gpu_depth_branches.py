"""GPU depth segmentation where it leaves its usual path: tiles with more distinct segment pairs than the boundary kernel's LDS
table takes (the rest goes to memory directly), and images more than 32767 pixels long (64-bit pixel offsets in the
assignment). Labels and boundary slots equal the oracle's; the boundary sums show in one step of a graph without edges, whose
every term is the boundary's or the prior's, at segment scales that are far from zero."""
import numpy as np
import pytest
import torch

from oracle import depth as D

pytestmark = pytest.mark.gpu

ds3 = pytest.importorskip("paper_2605_30488_amd.api")


def _noisy(H, W, rng, rough):
    v, u = np.mgrid[0:H, 0:W]
    z = 5.0 + np.sin(u / 7.0) + np.cos(v / 5.0) + rough * rng.normal(size=(H, W))
    x = np.stack([(u - W / 2) / W * z, (v - H / 2) / W * z, z], -1).astype(np.float32)
    x[rng.uniform(size=(H, W)) < 0.02] = 0.0
    return x, rng.uniform(1.3, 5.0, size=(H, W)).astype(np.float32)


def _check(H, W, M, rough, pairs_per_tile=0):
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(H + W)
    maps = [_noisy(H, W, rng, rough) for _ in range(2)]
    xyz, conf = [m[0] for m in maps], [m[1] for m in maps]
    a = ds3.build_arena(xyz, conf, "f32", dev)
    p = ds3.default_depth_params()
    p.segments_per_kf, p.min_seg_px = M, 1
    plan = ds3.DepthPlan(ds3.Graph(a, [], torch.zeros(1, dtype=torch.int32, device=dev), anchors=(0,)), p)
    prob = D.DepthProblem(xyz, conf, [], [], params=D.DepthParams(segments_per_kf=M, min_seg_px=1))
    assert len(prob.pairs) / 2 > 2 * pairs_per_tile   # unordered pairs of the two keyframes, a tile each
    lab = plan.labels().cpu().numpy()
    for k, (h, w, off) in enumerate(a.images):
        assert np.array_equal(lab[off:off + h * w], prob.glabel(k)), k
    assert plan.info["valid_segments"] == int(prob.seg_valid.sum())
    assert plan.info["boundary_slots"] == len(prob.pairs)
    eta0 = np.where(prob.seg_valid, rng.normal(size=prob.n_seg) * 0.05, 0.0)
    poses = np.zeros((2, 8))
    poses[:, 6:] = 1.0
    plan.set_eta(torch.as_tensor(eta0).to(dev))
    cost = plan.run(torch.as_tensor(poses).to(dev), 1).cpu().numpy()
    eta, ref = prob.run(poses, eta=eta0, iters=1)
    # a mean of differences held to 2^-41 each, with logarithms within 1e-14; a step is a weighted mean of such terms
    assert np.abs(eta - eta0).max() > 1e-3
    assert np.abs(plan.eta().cpu().numpy() - eta).max() <= 2e-12
    assert abs(cost[0] - ref[0]) <= 1e-9 * abs(ref[0])
    plan.close()


# 512 entries of the table, 16 probes; one tile of 64 x 32 pixels, whole and cut
@pytest.mark.parametrize("H,W,M,rough,pairs", [(32, 64, 200, 3.0, 550), (32, 64, 230, 8.0, 600), (31, 61, 200, 3.0, 520)])
def test_more_pairs_than_the_table(H, W, M, rough, pairs):
    _check(H, W, M, rough, pairs)


@pytest.mark.parametrize("H,W,M", [(4, 32767, 4), (4, 32769, 4), (33001, 5, 4), (3, 70001, 2)])
def test_long_images(H, W, M):
    _check(H, W, M, 0.5)
