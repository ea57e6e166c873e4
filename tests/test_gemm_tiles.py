"""bf16 products: the same bits whichever row tile a batch's size selects.  A few tasks of their own (small tiles) and the same
tasks at the head of a larger batch (larger tiles), rows and widths that are no multiples of a tile."""
from types import SimpleNamespace

import numpy as np
import pytest
import torch

from tests.test_gpu_parity import gm  # noqa: F401

pytestmark = pytest.mark.gpu
F, D, NDENSE, OWN = 4, 32, 5, 2048   # table rows of a task's own, half of them for each set


def _sets(sizes, which, F=F):
    """Every task draws from a generator of its own (task t is the same in every batch) and looks every row up once, so that a
    row's gradient is one sample's."""
    parts = []
    for t, n in enumerate(sizes):
        rng = np.random.default_rng([which, t])
        lens = rng.integers(1, 4, size=n * F)
        field = np.repeat(np.arange(n * F) % F, lens)
        idx = np.zeros(len(field), dtype=np.int64)
        for f in range(F):
            idx[field == f] = rng.permutation(OWN // 2)[:(field == f).sum()] + t * OWN + which * (OWN // 2)
        parts.append((lens, idx, rng.standard_normal((n, NDENSE)), rng.random(n) < 0.3))
    lens, idx, dense, labels = (np.concatenate(x) for x in zip(*parts))
    dev = "cuda:0"
    return SimpleNamespace(task_offsets=np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64),
                           bag_offsets=torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int64, device=dev),
                           indices=torch.tensor(idx, dtype=torch.int32, device=dev), dense=torch.tensor(dense, dtype=torch.float32, device=dev),
                           labels=torch.tensor(labels, dtype=torch.float32, device=dev))


@pytest.mark.parametrize("hidden,rows,many", [((264, 136), (201, 257), 150), ((264, 136), (101, 131), 90), ((512, 256), (256, 300), 140),
                                              ((1024, 264, 40), (195, 193), 70)])
@pytest.mark.parametrize("K", [1, 3])
def test_row_tiles(gm, hidden, rows, many, K):  # noqa: F811
    dims = [F * D + NDENSE, *hidden, 1]
    gen = torch.Generator("cuda").manual_seed(5)
    params = SimpleNamespace(emb=torch.randn(F * OWN * many, D, device="cuda", generator=gen) * 0.3,
                             W=[torch.randn(a, b, device="cuda", generator=gen) / a ** 0.5 for a, b in zip(dims[:-1], dims[1:])],
                             b=[torch.randn(b, device="cuda", generator=gen) * 0.1 for b in dims[1:]])
    got = []
    for T in (2, many):
        sizes = [rows[t % 2] for t in range(T)]
        ctx = gm(F, [OWN * many] * F, D, NDENSE, dims, 1, workspace_bytes=3 << 30)
        out = ctx.meta_step(_sets(sizes, 0), _sets(sizes, 1), params, 0.1, K, 2)
        n = int(out["n_emb_rows"].item())
        r = out["emb_rows"][:n]
        mine = r % (OWN * many) < 2 * OWN   # rows of the first two tasks
        got.append((out["task_loss"][:2].clone(), r[mine], out["emb_grad"][:n][mine]))
        ctx.close()
    assert len(got[0][1]) > 0 and float(got[0][2].abs().max()) > 0
    for a, b in zip(*got):
        assert torch.equal(a, b)


@pytest.mark.parametrize("K,order", [(1, 1), (3, 2)])
def test_forward_and_backward_tiles(gm, K, order):  # noqa: F811
    """Enough tasks that the products keep 256-row tiles: the same bits in 256 x 256 tiles as in 256 x 128 ones, with rows and contractions
    that are no multiples of a tile and tasks of one row."""
    f, T = 8, 150
    dims = [f * D + NDENSE, 512, 256, 1]
    gen = torch.Generator("cuda").manual_seed(8)
    params = SimpleNamespace(emb=torch.randn(f * OWN * T, D, device="cuda", generator=gen) * 0.3,
                             W=[torch.randn(a, b, device="cuda", generator=gen) / a ** 0.5 for a, b in zip(dims[:-1], dims[1:])],
                             b=[torch.randn(b, device="cuda", generator=gen) * 0.1 for b in dims[1:]])
    sup, qry = (_sets([(201, 257, 256, 1 + w, 480)[t % 5] for t in range(T)], w, f) for w in (0, 1))
    got = []
    for columns in (128, 256):
        ctx = gm(f, [OWN * T] * f, D, NDENSE, dims, 1, workspace_bytes=8 << 30)
        ctx.configure("gemm_tile_n", columns)
        out = ctx.meta_step(sup, qry, params, 0.1, K, order)
        n = int(out["n_emb_rows"].item())
        got.append([x.clone() for x in (out["task_loss"], *out["dW"], *out["db"], out["emb_grad"][:n])])
        ctx.close()
    assert float(got[0][-1].abs().max()) > 0
    for a, b in zip(*got):
        assert torch.equal(a, b)


@pytest.mark.parametrize("K", [1, 3, 4])
def test_weight_gradient_tiles(gm, K):  # noqa: F811
    """Tasks of about 200 rows under a first layer wide enough for 256 x 256 tiles of its gradients (remainders in both directions
    and in the contraction, single-row tasks among them): the same bits as in 128 x 128 tiles, one to four products a sum."""
    f, d, T = 8, 128, 110
    dims = [f * d + NDENSE, 256, 1]
    gen = torch.Generator("cuda").manual_seed(6)
    params = SimpleNamespace(emb=torch.randn(f * OWN * T, d, device="cuda", generator=gen) * 0.3,
                             W=[torch.randn(a, b, device="cuda", generator=gen) / a ** 0.5 for a, b in zip(dims[:-1], dims[1:])],
                             b=[torch.randn(b, device="cuda", generator=gen) * 0.1 for b in dims[1:]])
    sup, qry = (_sets([(193, 256, 257, 1 + w, 319)[t % 5] for t in range(T)], w, f) for w in (0, 1))
    got = []
    for wide in (1, 0):
        ctx = gm(f, [OWN * T] * f, d, NDENSE, dims, 1, workspace_bytes=8 << 30)
        ctx.configure("wgrad_wide", wide)
        out = ctx.meta_step(sup, qry, params, 0.1, K, 2)
        n = int(out["n_emb_rows"].item())
        got.append([x.clone() for x in (out["task_loss"], *out["dW"], *out["db"], out["emb_grad"][:n])])
        ctx.close()
    assert float(got[0][1].abs().max()) > 0
    for a, b in zip(*got):
        assert torch.equal(a, b)


def test_contraction_of_more_than_two_million(gm):  # noqa: F811
    """A hidden layer wider than 2^21 and no multiple of a tile's 64 contraction values, its backward product in 256 x 256 tiles: what lies
    past the last column counts as zero.  Only sixteen columns have weights: the last eight, and the eight of the last row that lie
    2^30 bytes behind the first row (an offset inside the tile, which once stood for "outside")."""
    wide, n, d = (1 << 21) + 32, 256, 64
    gen = torch.Generator("cuda").manual_seed(7)
    cols = torch.cat([torch.arange(8) + (1 << 29) % wide, torch.arange(8) + wide - 8]).cuda()
    w1 = torch.randn(F * d, 16, device="cuda", generator=gen) * 0.1
    params = SimpleNamespace(emb=torch.randn(F * n, d, device="cuda", generator=gen), W=[torch.zeros(F * d, wide, device="cuda"), torch.randn(wide, 1, device="cuda", generator=gen)],
                             b=[torch.zeros(wide, device="cuda"), torch.zeros(1, device="cuda")])
    params.W[0][:, cols] = w1
    y = (torch.arange(n, device="cuda") % 3 == 0).float()
    empty = SimpleNamespace(task_offsets=np.zeros(2, dtype=np.int64), bag_offsets=torch.zeros(1, dtype=torch.int64, device="cuda"),
                            indices=torch.zeros(0, dtype=torch.int32, device="cuda"), dense=torch.zeros(0, 0, device="cuda"), labels=torch.zeros(0, device="cuda"))
    query = SimpleNamespace(task_offsets=np.array([0, n], dtype=np.int64), bag_offsets=torch.arange(n * F + 1, dtype=torch.int64, device="cuda"),
                            indices=(torch.arange(n * F, device="cuda") // F).int(), dense=torch.zeros(n, 0, device="cuda"), labels=y)   # sample s: row s of every table
    ctx = gm(F, [n] * F, d, 0, [F * d, wide, 1], 1, workspace_bytes=52 << 30)
    out = ctx.meta_step(empty, query, params, 0.1, 0, 1)
    got = out["emb_grad"][:F * n].reshape(F, n, d).permute(1, 0, 2).reshape(n, F * d).clone()
    ctx.close()
    bf = lambda t: t.bfloat16().float()   # noqa: E731
    w, w2 = bf(w1), params.W[1][cols, 0]
    h = bf(torch.relu(bf(params.emb.reshape(F, n, d).permute(1, 0, 2).reshape(n, F * d)) @ w))
    delta = bf((torch.sigmoid(h @ w2) - y)[:, None] / n * w2 * (h > 0))
    want = delta @ w.T
    worst, largest = (got - want).norm(dim=1).max().item(), want.norm(dim=1).max().item()
    assert worst <= 2e-2 * largest and largest > 0
