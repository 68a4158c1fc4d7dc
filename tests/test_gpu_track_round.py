"""The tracker's two ways to run a round (one launch for few segments; a reduction and a step launch) give the same bits:
a call that records a timer takes two launches per round at any size. Sizes around a segment (4096 frame pixels), around
the step's staging of 64 segments, several problems in a call with one that has no matches, and 256 segments (the most
that take one launch) and 257."""
import numpy as np
import pytest
import torch

import oracle as O
from tests.helpers import exact_graph

pytestmark = pytest.mark.gpu

ds3 = pytest.importorskip("paper_2605_30488_amd.api")

SIZES = [[(9, 11)], [(64, 64)], [(17, 241)], [(512, 512)], [(520, 512)], [(9, 11), (17, 241), (64, 64), (130, 64)],
         [(512, 512)] * 4, [(512, 512)] * 3 + [(520, 512)]]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("frames", SIZES, ids=lambda f: f"{len(f)}x{f[-1][0]}x{f[-1][1]}")
def test_one_launch_rounds_match_two(frames, dtype):
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(7 + len(frames))
    xyz, conf, idx, T0 = [], [], [], []
    for p, (H, W) in enumerate(frames):
        x, c, _, ix, gt = exact_graph(n_kf=2, H=H, W=W, seed=100 + p, frac_valid=0.8)
        xyz += [np.asarray(v, np.float32) + rng.normal(size=np.shape(v)).astype(np.float32) * 1e-3 for v in x]
        conf += [np.asarray(v, np.float32) for v in c]
        m = np.asarray(ix[0]).reshape(-1).copy()
        if len(frames) > 1 and p == 1:
            m[:] = -1  # no matches at all
        idx.append(m)
        tau = np.concatenate([rng.normal(size=3) * 0.2, rng.normal(size=3) * 0.1, [0.05]])
        T0.append(O.sim3_update(gt[1][None], tau[None])[0])
    a = ds3.build_arena(xyz, conf, dtype, dev)
    ix = torch.as_tensor(np.concatenate(idx), dtype=torch.int32).to(dev)
    trk = ds3.Tracker(a, [(2 * p, 2 * p + 1) for p in range(len(frames))])
    out = []
    for timer in (ds3.KernelTimer(), None, None):  # the last: the round's tickets are back at zero
        T = torch.as_tensor(np.asarray(T0).reshape(-1, 8), dtype=torch.float64).to(dev)
        r = trk.run(ix, T, timer=timer)
        out.append([T.cpu().numpy()] + [v.cpu().numpy() for v in r])
    assert out[0][2].max() > 1
    for other in out[1:]:
        for u, v in zip(out[0], other):
            assert np.array_equal(u, v, equal_nan=u.dtype.kind == "f")
