"""GPU depth refinement at the edges of its tiles: the segmentation's (64 x 32 pixels per block, eight rows per thread, sums
per block; labels, segment counts and boundary table against the oracle's exact integer arithmetic) and the data term's
(64 x 64 pixels of keyframe j per block, 16 rows per wave, runs of one segment summed per lane), on rough pointmaps with
holes and low-confidence pixels so that members jump between cells and runs are short."""
import numpy as np
import pytest
import torch

import oracle as O
from oracle import depth as D

pytestmark = pytest.mark.gpu

ds3 = pytest.importorskip("paper_2605_30488_amd.api")


# one tile and a pixel less or more each way; a cell of one pixel; cells larger than a tile; several image shapes at once
def _rough(shapes):
    rng = np.random.default_rng(sum(h * w for h, w in shapes))
    xyz, conf = [], []
    for H, W in shapes:
        v, u = np.mgrid[0:H, 0:W]
        z = 5 + np.sin(u / 7.0) + np.cos(v / 5.0) + 0.05 * rng.normal(size=(H, W)) + 2.0 * (u > W // 2)
        x = np.stack([(u - W / 2) / W * z, (v - H / 2) / W * z, z], -1).astype(np.float32)
        x[rng.uniform(size=(H, W)) < 0.03] = 0.0
        xyz.append(x)
        conf.append(rng.uniform(1.3, 5, size=(H, W)).astype(np.float32))
    return rng, xyz, conf


@pytest.mark.parametrize("shapes,M", [([(32, 64)], 60), ([(31, 63)], 60), ([(33, 65)], 60), ([(8, 9)], 72),
                                      ([(100, 230)], 4), ([(65, 129), (33, 64), (7, 200)], 40)])
def test_labels_at_tile_edges(shapes, M):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    _, xyz, conf = _rough(shapes)
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


def _step_bound(prob, poses, eta, step):
    """First-order bound of a float32 data term's effect on each segment's step g / (1.05 H). With u = 2^-24, a match's
    products and sums are chains of at most 24 roundings, and r = s (sR x + t - b) has those of its terms, S = |s sR x| +
    |s t| + |s b| in place of |r|. So |dg| <= 24 u sum |w J| S and |dH| <= 24 u sum w J^2 S / max(|r|, kappa)."""
    H = prob.linearise(poses, eta)[1]
    dg, dH = np.zeros_like(H), np.zeros_like(H)
    for r, h, g, Jh, Jg in prob.residuals(poses, eta):
        a = np.abs(r)
        S = 2 * (np.abs(Jh) + np.abs(Jg)) + a          # |s t| <= |r| + |s sR x| + |s b|
        w = np.minimum(1.0, prob.P.huber_k / np.maximum(a, 1e-300))
        for seg, J in ((h, Jh), (g, Jg)):
            k = seg >= 0
            np.add.at(dg, seg[k], (w * np.abs(J) * S).sum(1)[k])
            np.add.at(dH, seg[k], (w * J * J * S / np.maximum(a, prob.P.huber_k)).sum(1)[k])
    return 24 * 2.0 ** -24 * (dg / 1.05 + np.abs(step) * dH) / H


# whole tiles, a pixel less or more each way, tiles with idle waves, thin images; matches clustered and scattered
@pytest.mark.parametrize("shape_i,shape_j", [((64, 64), (64, 64)), ((63, 65), (65, 63)), ((16, 200), (17, 129)),
                                             ((90, 70), (130, 9)), ((40, 64), (5, 70))])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_step_at_tile_edges(shape_i, shape_j, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    rng, xyz, conf = _rough([shape_i, shape_j])
    (Hi, Wi), (Hj, Wj) = shape_i, shape_j
    v, u = np.mgrid[0:Hj, 0:Wj]
    near = np.minimum(v, Hi - 1) * Wi + np.minimum(u + 1, Wi - 1)
    m = np.where(rng.uniform(size=(Hj, Wj)) < 0.1, rng.integers(0, Hi * Wi, size=(Hj, Wj)), near)
    idx = np.where(rng.uniform(size=(Hj, Wj)) < 0.8, m, -1).astype(np.int32).reshape(-1)
    poses = np.array([[0, 0, 0, 0, 0, 0, 1, 1], [0.02, -0.01, 0.03, 0.01, 0.02, -0.01, 0.99, 1.03]], np.float64)
    poses[1, 3:7] /= np.linalg.norm(poses[1, 3:7])
    a = ds3.build_arena(xyz, conf, dtype, dev)
    p = ds3.default_depth_params()
    p.segments_per_kf, p.min_seg_px = 40, 3
    plan = ds3.DepthPlan(ds3.Graph(a, [(0, 1)], torch.as_tensor(idx).to(dev), anchors=(0,)), p)
    if dtype == "bf16":
        xyz, conf = ([O.bf16_to_f32(O.bf16_round(x)).reshape(x.shape) for x in s] for s in (xyz, conf))
    prob = D.DepthProblem(xyz, conf, [(0, 1)], [idx], params=D.DepthParams(segments_per_kf=40, min_seg_px=3))
    eta0 = np.where(prob.seg_valid, rng.normal(size=prob.n_seg) * 0.05, 0.0)
    plan.set_eta(torch.as_tensor(eta0).to(dev))
    cost = plan.run(torch.as_tensor(poses).to(dev), 1).cpu().numpy()
    eta, ref = prob.run(poses, eta=eta0, iters=1)
    # 1e-13: float64 sums in another order; an anchor's segments do not move
    assert np.all(np.abs(plan.eta().cpu().numpy() - eta) <= _step_bound(prob, poses, eta0, eta - eta0) + 1e-13)
    assert np.max(np.abs(cost - ref) / np.abs(ref)) <= 1e-5
    plan.close()
