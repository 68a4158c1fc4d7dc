"""The batched matching's split into strips and runs, and references of more than 2^24 pixels.

The batched kernels give several strips of queries (and several runs of the mutual check) to a block once a call is large,
over directions of mixed sizes laid end to end: every edge is compared bit for bit with the call for one edge, whose
kernels take one run per block and their tables as arguments, and small edges with the oracle. An image of more than 2^24
pixels is a smooth scene in its last corner and holes elsewhere, with the queries one pixel aside: the match of a pixel is
its neighbour."""
import numpy as np
import pytest
import torch

import oracle as O

pytestmark = pytest.mark.gpu

ds3 = pytest.importorskip("paper_2605_30488_amd.api")


def _surface(u, v, H, W):
    x, y = (u - 0.5 * W) / max(H, W), (v - 0.5 * H) / max(H, W)
    d = 2.0 + 0.3 * torch.sin(3 * x) + 0.2 * torch.cos(4 * y)
    return torch.stack([x * d, y * d, d], -1)


def _map(H, W, rng, du=0.0, dv=0.0, grid=None):
    """xyz and confidence of every pixel of an H x W image that sees the surface of `grid` at its own place + (du, dv)."""
    Hr, Wr = grid or (H, W)
    v, u = torch.meshgrid(torch.arange(H, dtype=torch.float64), torch.arange(W, dtype=torch.float64), indexing="ij")
    X = _surface(u * (Wr - 1) / max(W - 1, 1) + du, v * (Hr - 1) / max(H - 1, 1) + dv, Hr, Wr).reshape(-1, 3)
    X[torch.as_tensor(rng.random(H * W) < 0.02)] = 0.0
    c = torch.as_tensor(rng.uniform(0.05, 3.0, H * W))
    return X.float(), c.float()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n_edges", [3, 12, 26, 92])
def test_batch_equals_single_edges(n_edges, dtype):
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(n_edges)
    sizes = [(384, 512), (33, 70), (384, 512), (16, 16), (2, 3), (101, 257)]
    maps = [_map(H, W, rng) for H, W in sizes]
    arena = ds3.build_arena([m[0].numpy().reshape(H, W, 3) for m, (H, W) in zip(maps, sizes)],
                            [m[1].numpy().reshape(H, W) for m, (H, W) in zip(maps, sizes)], dtype, dev)
    small = [(1, 3), (4, 1), (5, 3), (0, 1), (3, 5)]
    edges = [small[e] if e < len(small) and n_edges > 3 else ((0, 2), (2, 0), (5, 1))[e % 3] if n_edges == 3 else
             ((0, 2), (2, 0))[e % 2] for e in range(n_edges)]
    cross, off, idx_off, at = [], [], [], 0
    for i, j in edges:
        for a, b in ((j, i), (i, j)):
            X, c = _map(*sizes[a], rng, du=rng.uniform(-3, 3), dv=rng.uniform(-3, 3), grid=sizes[b])
            cross.append(ds3.pack_xyzc(X.to(dev), c.to(dev), dtype))
            off.append(at)
            at += len(X)
        idx_off.append(sum(sizes[b][0] * sizes[b][1] for _, b in edges[:len(idx_off)]))
    total = idx_off[-1] + sizes[edges[-1][1]][0] * sizes[edges[-1][1]][1]
    steps = torch.zeros(1, dtype=torch.int64, device=dev)
    idx, valid, nu, admit = ds3.match_batch(arena, torch.cat(cross), off, edges, idx_off, total, lm_steps=steps)
    assert steps.item() > 0
    part = [arena.data[o:o + H * W] for H, W, o in arena.images]
    for e, (i, j) in enumerate(edges):
        one = ds3.match_bidir(part[i], cross[2 * e], part[j], cross[2 * e + 1], sizes[i], sizes[j], dtype)
        sl = slice(idx_off[e], idx_off[e] + sizes[j][0] * sizes[j][1])
        assert torch.equal(one[0], idx[sl]) and torch.equal(one[1], valid[sl]), (e, i, j)
        assert torch.equal(one[2], nu[e]) and one[3].item() == admit[e].item()
        if max(sizes[i][0], sizes[j][0]) <= 101 and dtype == "f32":
            h = [t.cpu().numpy().astype(np.float64) for t in (part[i], cross[2 * e], part[j], cross[2 * e + 1])]
            s = [sizes[i], sizes[j], sizes[j], sizes[i]]
            X = [a[:, :3].reshape(*n, 3) for a, n in zip(h, s)]
            r = O.match_bidir(X[0], X[1], X[2], X[3], h[0][:, 3].reshape(sizes[i]), h[2][:, 3].reshape(sizes[j]))
            got = idx[sl].cpu().numpy()
            either = (r.idx_j2i.reshape(-1) >= 0) | (got >= 0)
            assert (r.idx_j2i.reshape(-1) == got)[either].mean() >= 0.98 if either.any() else True


@pytest.mark.parametrize("H,W", [(4096, 4096), (4096, 4097), (4300, 4099)])
def test_reference_around_2_24_pixels(H, W):
    dev = torch.device("cuda:0")
    h, w = 40, 48
    X, _ = _map(h, w, np.random.default_rng(3))
    X = X.reshape(h, w, 3).to(dev)
    ref = torch.zeros((H, W, 4), dtype=torch.float32, device=dev)
    ref[H - h:, W - w:, :3] = X
    ref[..., 3] = 1.0
    qry = torch.zeros_like(ref)
    qry[H - h:, W - w:W - 1, :3] = X[:, 1:]  # a pixel holds its right neighbour's point
    got = ds3.match(ref.reshape(-1, 4), (H, W), qry.reshape(-1, 4), (H, W)).reshape(H, W)
    assert (got[:H - h] == -1).all() and (got[:, :W - w] == -1).all()
    live = (X[..., 2] > 0).float()[None, None]
    # pixels whose cells, from their own to their neighbour's, hold no hole
    ok = -torch.nn.functional.max_pool2d(-torch.nn.functional.pad(live, (2, 2, 2, 2)), 5, 1)[0, 0] > 0
    ok[:, -3:] = False
    assert ok.sum() > 200
    n = torch.arange(H * W, device=dev, dtype=torch.int32).reshape(H, W)[H - h:, W - w:]
    assert torch.equal(got[H - h:, W - w:][ok], (n + 1)[ok])
