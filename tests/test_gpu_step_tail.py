"""The plain step ends in one launch (the ladder's attempts after the first, the update, the cost): against the same step
made of its parts, gn_linearize, chol_ladder_solve and sim3_update, which have launches of their own. One, two, three and nine
tiles of the solver; attempt 0 succeeding, a later attempt succeeding (lambda = -2 makes the system negative definite until
eps outgrows it), every attempt failing, and a single attempt. Solution, status and cost are the same numbers; the
poses go through the same operations in another kernel, where a product may be fused into a sum: a few rounding
errors of values below 10."""
import numpy as np
import pytest
import torch

from tests.helpers import exact_graph, perturb

pytestmark = pytest.mark.gpu

ds3 = pytest.importorskip("paper_2605_30488_amd.api")


@pytest.mark.parametrize("lam,mult,attempts", [(0.0, 100.0, 6), (-2.0, 1e6, 6), (-2.0, 1.0, 4), (-2.0, 100.0, 1)])
@pytest.mark.parametrize("n_kf", [2, 6, 12, 40])
def test_step_equals_its_parts(n_kf, lam, mult, attempts):
    dev = torch.device("cuda:0")
    edges = [(k, k + 1) for k in range(n_kf - 1)] + [(k, k + 3) for k in range(n_kf - 3)]
    xyz, conf, edges, idx, gt = exact_graph(n_kf=n_kf, H=8, W=12, seed=5, edges=edges, frac_valid=0.8)
    a = ds3.build_arena([np.asarray(x, np.float32) for x in xyz], [np.asarray(c, np.float32) for c in conf], "f32", dev)
    flat = torch.as_tensor(np.concatenate([np.asarray(v).reshape(-1) for v in idx]), dtype=torch.int32).to(dev)
    G = ds3.Graph(a, edges, flat, [96 * e for e in range(len(edges))], anchors=(0,))
    P = torch.as_tensor(perturb(gt, np.random.default_rng(6), rot=0.01, trans=0.01, scale=0.01, fixed=(0,))).to(dev)
    prm = ds3.default_gn_params()
    prm.lam = lam
    prm.eps_mult, prm.max_attempts = mult, attempts
    H, g, cost, _ = ds3.gn_linearize(G, P, prm)
    tau, st = ds3.chol_ladder_solve(H, g, lam, prm.eps0, mult, attempts)
    if lam == 0.0:
        assert st.item() == 0
    elif mult > 100.0:
        assert st.item() > 0
    else:
        assert st.item() == -1 and not tau.any()
    want = P.clone()
    fixed = torch.zeros(n_kf, dtype=torch.uint8, device=dev)
    fixed[0] = 1
    ds3.sim3_update(want, tau, fixed)
    for _ in range(2):
        got = P.clone()
        c, s, t = ds3.sim3_gn_step(G, got, prm, want_tau=True)
        assert s.item() == st.item() and torch.equal(t, tau) and c.item() == cost.item()
        assert float((got - want).abs().max()) <= 16 * 10 * 2.0 ** -52
        assert torch.equal(got[0], P[0])
