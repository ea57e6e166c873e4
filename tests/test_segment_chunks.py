"""The sparse gradient's sums over short lists of narrow rows: lists whose partial rows leave room for chunks of 16, of 32 (one
field, about 20000 lookups of 16 columns), and lists beyond 32768 lookups, in chunks of 64; row-list and table-shaped output."""
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
