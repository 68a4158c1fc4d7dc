"""Gradients of the cost where many matches share a pixel of the gathered keyframe: a wave's 64 gradients pass between its lanes
through LDS before they are added, twice per thread and tile. One pixel for all, a handful within a wave, every second match
missing, holes on both sides; against the FP64 oracle. The matches are wrong by metres, so that residuals are far from
cancellation and float32 resolves every channel."""
import numpy as np
import pytest
import torch

import oracle as O
from tests.helpers import exact_graph, perturb, pixel_channel_err, tangent_group_err

pytestmark = pytest.mark.gpu

ds3 = pytest.importorskip("paper_2605_30488_amd.api")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("hw", [(5, 13), (16, 32), (31, 35)])
@pytest.mark.parametrize("pool,frac", [(1, 1.0), (5, 1.0), (64, 0.5)])
def test_gradients_of_shared_pixels(hw, pool, frac, dtype):
    dev = torch.device("cuda:0")
    H, W = hw
    rng = np.random.default_rng(H * W + pool)
    xyz, conf, edges, idx, gt = exact_graph(n_kf=3, H=H, W=W, seed=H + pool)
    idx = [np.where(rng.random(H * W) < frac, rng.choice(rng.integers(0, H * W, pool), H * W), -1).astype(np.int32)
           for _ in idx]
    xyz = [np.where(rng.random((H, W, 1)) < 0.03, 0.0, x).astype(np.float32) for x in xyz]
    conf = [np.asarray(c, np.float32) for c in conf]
    poses = perturb(gt, rng, rot=0.05, trans=0.1, scale=0.05, fixed=())
    a = ds3.build_arena(xyz, conf, dtype, dev)
    G = ds3.Graph(a, edges, torch.as_tensor(np.concatenate(idx)).to(dev), anchors=(0,))
    gx, gc, gtau = ds3.gn_cost_adjoint(G, torch.as_tensor(poses).to(dev))
    if dtype == "bf16":
        xyz, conf = ([O.bf16_to_f32(O.bf16_round(v)).reshape(v.shape) for v in s] for s in (xyz, conf))
    _, rx, rc, rt = O.cost_grad(O.Graph(xyz, conf, edges, idx, anchors=()), poses)
    off = np.cumsum([0] + [H * W] * 3)
    assert pixel_channel_err(gx.cpu().numpy(), rx, off) <= 2e-4
    assert pixel_channel_err(gc.cpu().numpy(), rc, off) <= 2e-4
    assert tangent_group_err(gtau.cpu().numpy(), rt) <= 1e-3
