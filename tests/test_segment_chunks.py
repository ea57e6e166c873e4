"""The sparse gradient's sums over short lists of narrow rows: lists whose partial rows leave room for chunks of 16, of 32 (one
field, about 20000 lookups of 16 columns), and lists beyond 32768 lookups, in chunks of 64; row-list and table-shaped output."""
from types import SimpleNamespace

import numpy as np
import pytest
import torch

from tests.helpers import small_cfg
from tests.test_gpu_parity import TOL_FP32, _compare_step, _inputs, _params_dev, _to_dev, gm  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tasks,rows", [(2, 300), (8, 500), (16, 512)])
def test_chunk_lengths(gm, tasks, rows):  # noqa: F811
    cfg = small_cfg(n_tasks=tasks, n_fields=1, emb_dim=16, rows_per_field=900, n_support=rows, n_query=rows, layer_dims=(21, 8, 1))
    sup, qry, params = _inputs(cfg, emb_std=0.3)
    n = sup.indices.numel() + qry.indices.numel()
    assert {2: n < 8192, 8: 16384 < n < 32768, 16: n > 32768}[tasks]
    ctx = gm.from_config(cfg, workspace_bytes=1 << 28)
    _compare_step(cfg, ctx, sup, qry, params, 1, 2, TOL_FP32, f"{n} lookups")
    ds, dq, dp = _to_dev(sup, ctx.device), _to_dev(qry, ctx.device), _params_dev(params, ctx.device)
    out = ctx.meta_step(ds, dq, dp, cfg.inner_lr, 1, 2)
    table = torch.zeros_like(dp.emb)
    ctx.meta_step(ds, dq, dp, cfg.inner_lr, 1, 2, emb_grad_table=table)
    m = int(out["n_emb_rows"].item())
    assert torch.equal(table[out["emb_rows"][:m]], out["emb_grad"][:m]), "the same chunks either way"
    ctx.close()


@pytest.mark.parametrize("dim,n_rows,tasks", [(4, 2, 3), (16, 3, 40), (64, 3, 12), (64, 37, 64), (256, 2, 6)])
def test_long_segments(gm, dim, n_rows, tasks):  # noqa: F811
    """Few rows with thousands of lookups each: segments of more pieces than a lane group adds by itself, a round of the
    workgroup's and the next one, more of them than its list holds or none, in both shapes of the output."""
    cfg = small_cfg(n_tasks=tasks, n_fields=2, emb_dim=dim, rows_per_field=n_rows, n_support=96, n_query=104, bag_max=9,
                    layer_dims=(2 * dim + 5, 8, 1))
    sup, qry, params = _inputs(cfg, emb_std=0.3)
    ctx = gm.from_config(cfg, workspace_bytes=1 << 30)
    _compare_step(cfg, ctx, sup, qry, params, 0, 1, TOL_FP32, f"{tasks} tasks, {n_rows} rows of {dim}")
    ds, dq, dp = _to_dev(sup, ctx.device), _to_dev(qry, ctx.device), _params_dev(params, ctx.device)
    out = ctx.meta_step(ds, dq, dp, cfg.inner_lr, 0, 1)
    table = torch.zeros_like(dp.emb)
    ctx.meta_step(ds, dq, dp, cfg.inner_lr, 0, 1, emb_grad_table=table)
    m = int(out["n_emb_rows"].item())
    assert torch.equal(table[out["emb_rows"][:m]], out["emb_grad"][:m]), "the same order either way"
    ctx.close()


@pytest.mark.parametrize("dim,fields,lookups,mode", [(32, 3, (1 << 22) + 4097, "plain"), (64, 2, (1 << 22) + 255, "ordered"), (128, 1, 1 << 22, "plain"),
                                                     (64, 2, (1 << 22) - 1, "ordered")])
def test_chunks_inside_long_segments(gm, dim, fields, lookups, mode):  # noqa: F811
    """Lists long enough for the chunks inside long segments to be taken in another order (and one just too short): a row with a
    quarter of a field's lookups, some of thousands, rows of one, a last block that is not full; values in both forms.  A row's sum is
    64 terms a chunk and then its chunks one after the other, so it is off by at most that many roundings of the sum of magnitudes."""
    T, R, samples = 150 // fields, 5_000, 512
    gen = torch.Generator().manual_seed(dim)
    n = lookups // 2

    def some(n):
        off = torch.cat([torch.zeros(1, dtype=torch.int64), torch.randint(0, n + 1, (T * samples * fields - 1,), generator=gen).sort().values, torch.full((1,), n)])
        idx = (torch.rand(n, generator=gen) ** 6 * R).int().clamp(max=R - 1)
        idx[torch.rand(n, generator=gen) < 0.25] = 7
        return SimpleNamespace(task_offsets=np.arange(T + 1, dtype=np.int64) * samples, bag_offsets=off.cuda(), indices=idx.cuda(),
                               dense=torch.randn(T * samples, 1, generator=gen).cuda(), labels=(torch.rand(T * samples, generator=gen) < 0.3).float().cuda())
    sup, qry = some(lookups - n), some(n)
    W = torch.randn(fields * dim + 1, 1, generator=gen).cuda() / dim
    params = SimpleNamespace(emb=torch.randn(fields * R, dim, generator=gen).cuda() * 0.01, W=[W], b=[torch.zeros(1, device="cuda")])
    ctx = gm(fields, [R] * fields, dim, 1, [fields * dim + 1, 1], 0, workspace_bytes=6 << 30)
    if mode == "plain":
        ctx.configure("adapt_rows", 0)
    else:
        ctx.configure("index_path", 2)
    out = ctx.meta_step(sup, qry, params, 0.1, 0 if mode == "plain" else 1, 1)
    m = int(out["n_emb_rows"].item())
    got = torch.zeros(fields * R, dim, dtype=torch.float64, device="cuda")
    got[out["emb_rows"][:m]] = out["emb_grad"][:m].double()
    table = torch.zeros_like(params.emb)
    ctx.meta_step(sup, qry, params, 0.1, 0 if mode == "plain" else 1, 1, emb_grad_table=table)
    ctx.close()
    assert torch.equal(table.double(), got)

    def pool(s, emb):
        bag = torch.repeat_interleave(torch.arange(T * samples * fields, device="cuda"), s.bag_offsets.diff())
        row = s.indices.long() + bag % fields * R
        return bag, row, torch.zeros(T * samples * fields, dim, dtype=torch.float64, device="cuda").index_add_(0, bag, emb[row])
    emb, w, b = params.emb.double(), W.double().repeat(1, T).T.contiguous(), torch.zeros(T, dtype=torch.float64, device="cuda")
    task = torch.arange(T * samples, device="cuda") // samples
    if mode == "ordered":   # one inner step: a task's rows, weights and bias
        bag, row, x = pool(sup, emb)
        x = torch.cat([x.view(T * samples, -1), sup.dense.double()], 1)
        dz = (torch.sigmoid((x * w[task]).sum(1)) - sup.labels.double()) / samples
        w1 = w - 0.1 * torch.zeros_like(w).index_add_(0, task, dz[:, None] * x)
        b = b - 0.1 * torch.zeros_like(b).index_add_(0, task, dz)
        dx = (dz[:, None] * w[task])[:, :-1].reshape(T * samples * fields, dim)
        cell = task[bag // fields] * (fields * R) + row
        own = torch.zeros(T * fields * R, dim, dtype=torch.float64, device="cuda").index_add_(0, cell, dx[bag])
        own = emb.repeat(T, 1) - 0.1 * own
        bag, row, _ = pool(qry, emb)
        xq = torch.zeros(T * samples * fields, dim, dtype=torch.float64, device="cuda").index_add_(0, bag, own[task[bag // fields] * (fields * R) + row])
        w = w1
    else:
        bag, row, xq = pool(qry, emb)
    xq = torch.cat([xq.view(T * samples, -1), qry.dense.double()], 1)
    dz = (torch.sigmoid((xq * w[task]).sum(1) + b[task]) - qry.labels.double()) / samples
    dx = (dz[:, None] * w[task])[:, :-1].reshape(T * samples * fields, dim)
    want = torch.zeros_like(got).index_add_(0, row, dx[bag])
    size = torch.zeros_like(got).index_add_(0, row, dx[bag].abs())
    scale = float((got * want).sum() / (want * want).sum())
    assert abs(scale * T - 1) < 1e-4 or abs(scale - 1) < 1e-4    # (a mean or a sum over the tasks)
    terms = 64 + torch.bincount(row, minlength=fields * R).max().item() / 64 + 8 * dim * fields   # (.. and the logit's own terms)
    assert bool(((got / scale - want).abs() <= terms * 2.0 ** -24 * size + 1e-12).all())


@pytest.mark.parametrize("dim,tasks", [(16, 4), (64, 40)])
@pytest.mark.parametrize("K,order", [(0, 2), (2, 1)])
def test_no_query_rows(gm, dim, tasks, K, order):  # noqa: F811
    """Without a chain the support set's lookups have zero gradients, which are not read; with nothing else in the batch they are written."""
    cfg = small_cfg(n_tasks=tasks, n_fields=2, emb_dim=dim, rows_per_field=50, n_support=30, n_query=4, layer_dims=(2 * dim + 5, 8, 1))
    sup, _, params = _inputs(cfg, emb_std=0.3)
    ctx = gm.from_config(cfg, workspace_bytes=1 << 29)
    ds, dp = _to_dev(sup, ctx.device), _params_dev(params, ctx.device)
    none = SimpleNamespace(task_offsets=np.zeros(tasks + 1, dtype=np.int64), bag_offsets=torch.zeros(1, dtype=torch.int64, device="cuda"), labels=ds.labels[:0],
                           indices=ds.indices[:0], dense=ds.dense[:0])
    for table in (None, torch.ones_like(dp.emb)):
        out = ctx.meta_step(ds, none, dp, cfg.inner_lr, K, order, emb_grad_table=table)
        if table is None:
            n = int(out["n_emb_rows"].item())
            assert n > 0 and not out["emb_grad"][:n].any()
        else:
            assert torch.equal(table, torch.ones_like(table))
    ctx.close()
