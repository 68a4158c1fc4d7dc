"""The match-stream reduction of 16-byte (bfloat16) records at the edges of its groups: whole groups of 256 U records go
without a compare per record, the rest with one. A record meets the same thread in the same order whatever U is, so the sums
have the same bits for one, two and four records in flight; the count is exact; and the cost agrees with the plain form,
which adds the same non-negative terms in another order: at most 32 roundings on either side."""
import numpy as np
import pytest
import torch

from tests.helpers import exact_graph, perturb

pytestmark = pytest.mark.gpu

ds3 = pytest.importorskip("paper_2605_30488_amd.api")


@pytest.mark.parametrize("H", [64, 65])
@pytest.mark.parametrize("n", [0, 1, 255, 256, 257, 511, 512, 513, 1023, 1024, 1025, 2048, 3000, 4096])
def test_group_edges(n, H):
    dev = torch.device("cuda:0")
    W = 64
    xyz, conf, edges, idx, gt = exact_graph(n_kf=2, H=H, W=W, seed=3, frac_valid=1.0)
    rng = np.random.default_rng(n)
    m = np.asarray(idx[0]).reshape(-1).copy()
    m[rng.permutation(H * W)[n:]] = -1  # n matches, anywhere in the image
    a = ds3.build_arena([np.asarray(x, np.float32) for x in xyz], [np.asarray(c, np.float32) for c in conf], "bf16", dev)
    G = ds3.Graph(a, edges, torch.as_tensor(m, dtype=torch.int32).to(dev), [0], anchors=(0,))
    P = torch.as_tensor(perturb(gt, np.random.default_rng(1), rot=0.01, trans=0.01, scale=0.01, fixed=(0,))).to(dev)
    out = []
    for unroll in (1, 2, 4):
        Q = P.clone()
        plan = ds3.GNPlan(G, Q, px_per_thread=16, unroll=unroll)
        cost, st = plan.run(2)
        out.append((cost.cpu(), st.cpu(), Q.cpu()))
        plan.close()
    for other in out[1:]:
        assert all(torch.equal(x, y) for x, y in zip(out[0], other))
    _, _, plain, count = ds3.gn_linearize(G, P)
    assert count.item() <= n and (n == 0 or count.item() >= 0.9 * n)
    assert abs(out[0][0][0].item() - plain.item()) <= 64 * 2.0 ** -24 * plain.item()
