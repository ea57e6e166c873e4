"""The row hops at the edges of their tiles: task sizes around 64, 128 and 256 rows in either set, tasks with an empty
support set, more than eight tasks (the lists of the XCDs), one and two column tiles per row and rows of several slices,
tasks of up to 1024 rows (four tiles and a run of fields beyond the first)."""
import dataclasses

import numpy as np
import pytest
import torch

from tests.helpers import small_cfg
from tests.test_gpu_parity import TOL_FP32, _compare_step, _inputs, _params_dev, _to_dev, gm  # noqa: F401

pytestmark = pytest.mark.gpu


def _cut(s, sizes, F):
    """The first sizes[t] samples of every task."""
    keep = np.concatenate([np.arange(a, a + n) for a, n in zip(s.task_offsets[:-1], sizes)]).astype(np.int64)
    off = s.bag_offsets.numpy()
    lens = off[1:] - off[:-1]
    bags = (keep[:, None] * F + np.arange(F)).reshape(-1)
    idx = np.concatenate([np.arange(off[b], off[b + 1]) for b in bags]) if len(bags) else np.zeros(0, np.int64)
    return dataclasses.replace(s, task_offsets=np.concatenate([[0], np.cumsum(sizes)]).astype(s.task_offsets.dtype),
                               bag_offsets=torch.from_numpy(np.concatenate([[0], np.cumsum(lens[bags])])), indices=s.indices[torch.from_numpy(idx)],
                               dense=s.dense[torch.from_numpy(keep)], labels=s.labels[torch.from_numpy(keep)])


@pytest.mark.parametrize("F,D,bf,ns,nq", [
    (3, 64, 0, [1, 64, 63, 64, 32, 33, 2, 31, 7, 64], [64, 1, 63, 64, 33, 32, 2, 31, 64, 64]),
    (3, 64, 0, [65, 64, 128, 129, 1, 192, 3, 66, 127, 193], [64, 65, 129, 128, 193, 1, 128, 3, 66, 127]),
    (3, 32, 0, [257, 10, 256, 255, 64, 65, 300, 130], [10, 257, 255, 256, 65, 64, 130, 300]),
    (3, 128, 0, [70, 5, 200], [5, 70, 129]),
    (3, 64, 1, [320, 64, 65, 9, 40], [33, 64, 257, 130, 40]),
    (9, 32, 0, [513, 30, 1024, 769, 200], [1024, 31, 513, 100, 768]),
    (9, 32, 0, [512, 1024, 449, 768, 448, 256], [768, 256, 512, 450, 512, 512])])   # (tiles of equal height first; not with 448 rows)
def test_tile_edges(gm, F, D, bf, ns, nq):  # noqa: F811
    cfg = small_cfg(n_tasks=len(ns), n_fields=F, emb_dim=D, rows_per_field=60, n_support=max(ns), n_query=max(nq), bag_max=3 if F < 9 else 1,
                    layer_dims=(F * D + 5, 40, 1), mlp_dtype=bf)
    sup, qry, params = _inputs(cfg, emb_std=0.3)
    sup, qry = _cut(sup, ns, F), _cut(qry, nq, F)
    ctx = gm.from_config(cfg, workspace_bytes=1 << 29)
    ctx.configure("row_path", 2)
    _compare_step(cfg, ctx, sup, qry, params, 2, 2, 2e-2 if bf else TOL_FP32, f"rows of {D}, {ns} / {nq}", operand="bf16" if bf else "fp64")
    ctx.close()


@pytest.mark.parametrize("tasks,fields", [(2, 17), (64, 3)])   # runs of eight fields with one left over; the first batch dealt by whole tasks
def test_runs_of_fields(gm, tasks, fields):  # noqa: F811
    cfg = small_cfg(n_tasks=tasks, n_fields=fields, emb_dim=32, rows_per_field=60, n_support=66, n_query=65, bag_max=2,
                    layer_dims=(fields * 32 + 5, 24, 1))
    sup, qry, params = _inputs(cfg, emb_std=0.3)
    ctx = gm.from_config(cfg, workspace_bytes=1 << 29)
    ctx.configure("row_path", 2)
    _compare_step(cfg, ctx, sup, qry, params, 2, 2, TOL_FP32, f"{tasks} tasks x {fields} fields")
    ctx.close()


@pytest.mark.parametrize("rows,samples,bag,zipf", [(64, 120, 8, 0.0), (65, 200, 6, 0.0), (130, 256, 9, 0.0), (129, 300, 9, 0.0), (700, 512, 12, 1.05),
                                                   (5000, 250, 20, 0.6), (33, 700, 3, 0.0)])
@pytest.mark.parametrize("K", [1, 2])
def test_batches_of_hot_rows(gm, rows, samples, bag, zipf, K):  # noqa: F811
    """Rows that both sets look up often: one batch of the counting kernel exactly full, one row over, several batches and tiles
    of out-rows, more distinct rows than a workgroup has threads, sets of more than 512 samples."""
    cfg = small_cfg(n_tasks=3, n_fields=2, emb_dim=32, rows_per_field=rows, n_support=samples, n_query=samples - 30, bag_max=bag, zipf_s=zipf,
                    layer_dims=(2 * 32 + 5, 24, 1))
    sup, qry, params = _inputs(cfg, emb_std=0.3)
    ctx = gm.from_config(cfg, workspace_bytes=1 << 29)
    ctx.configure("row_path", 2)
    _compare_step(cfg, ctx, sup, qry, params, K, 2, TOL_FP32, f"{rows} rows, {samples} samples, bags of {bag}")
    ctx.close()


@pytest.mark.parametrize("large,bag,matrices", [((600,), 12, True), ((1024, 513), 12, True), ((1025, 600), 12, None), ((600,), 3, False),
                                                ((1024, 1024, 1024), 12, True), ((1024,) * 6, 12, False)])
def test_few_large_tasks_among_small_ones(gm, large, bag, matrices):  # noqa: F811
    """Tasks of more than 512 rows take the others' matrices where they are few and lookups many: then the bits are those of matrices
    for all (matrices: True), else another order of sums; never more than rounding away from the sparse kernel's."""
    F, D = 3, 32
    sizes = [*large, *([200, 250, 193] * 29)]
    cfg = small_cfg(n_tasks=len(sizes), n_fields=F, emb_dim=D, rows_per_field=500, n_support=max(sizes), n_query=max(sizes), bag_max=bag,
                    layer_dims=(F * D + 5, 24, 1))
    sup, qry, params = _inputs(cfg, emb_std=0.3)
    ctx = gm.from_config(cfg, workspace_bytes=1 << 31)
    s, q, p = _to_dev(_cut(sup, sizes, F), ctx.device), _to_dev(_cut(qry, sizes, F), ctx.device), _params_dev(params, ctx.device)
    got = {}
    for path in (0, 1, 2):
        if path == 2 and max(sizes) > 1024:
            continue
        ctx.configure("row_path", path)
        out = ctx.meta_step(s, q, p, cfg.inner_lr, 2, 2)
        n = int(out["n_emb_rows"].item())
        got[path] = [x.clone() for x in (out["emb_grad"][:n], out["task_loss"][:len(sizes)], *out["dW"])]
    ctx.close()
    for a, b in zip(got[0], got[1]):
        assert float((a - b).norm()) <= TOL_FP32 * float(b.norm())
    if matrices is not None:
        same = all(torch.equal(a, b) for a, b in zip(got[0], got[2]))
        assert same == matrices


def _few_large(fields):
    sizes = [1024, 600, *([200, 250, 193] * 29)]
    cfg = small_cfg(n_tasks=len(sizes), n_fields=fields, emb_dim=32, rows_per_field=500, n_support=max(sizes), n_query=max(sizes), bag_max=12,
                    layer_dims=(fields * 32 + 5, 24, 1))
    sup, qry, params = _inputs(cfg, emb_std=0.3)
    return cfg, _cut(sup, sizes, fields), _cut(qry, sizes, fields), params


def test_few_large_tasks_in_any_workspace(gm):  # noqa: F811
    """The batch alone decides how a few large tasks' rows are summed: losses and row gradients are the same bits in every workspace,
    however many waves it takes, and whether training iterations overlap with both batches' matrices in place, one batch's, or not at all."""
    cfg, sup, qry, params = _few_large(3)
    dev = torch.device("cuda", 0)
    s, q, want = _to_dev(sup, dev), _to_dev(qry, dev), None
    for mib in [1024, *range(420, 110, -12)]:
        ctx = gm.from_config(cfg, workspace_bytes=mib << 20)
        p = _params_dev(params, dev)
        out = ctx.meta_step(s, q, p, cfg.inner_lr, 2, 2)
        n = int(out["n_emb_rows"].item())
        got = [out["emb_rows"][:n].clone(), out["emb_grad"][:n].clone(), out["task_loss"][:cfg.n_tasks].clone()]
        want = want or got
        assert all(torch.equal(a, b) for a, b in zip(got, want)), f"{mib} MiB"
        one, loop = _params_dev(params, dev), _params_dev(params, dev)
        for _ in range(2):
            ctx.meta_train_step(s, q, one, cfg.inner_lr, 2, 2, 0.01)
        ctx.meta_train([(s, q)] * 2, loop, cfg.inner_lr, 2, 2, 0.01)
        ctx.close()
        assert all(torch.equal(a, b) for a, b in zip([one.emb, *one.W, *one.b], [loop.emb, *loop.W, *loop.b])), f"{mib} MiB"


def test_loop_stops_at_a_batch_beyond_the_matrices(gm):  # noqa: F811
    """Matrices forced, a batch beyond their limits after a good one: with both batches' matrices in place, one batch's, or no overlap, the
    good iteration is applied and the other is not."""
    from paper_2401_04338_amd import GMetaError
    dev = torch.device("cuda", 0)
    sets = []
    for bag in (12, 200):   # (a matrix takes bags of at most 127)
        cfg = small_cfg(n_tasks=20, n_fields=3, emb_dim=32, rows_per_field=500, n_support=500, n_query=500, bag_max=12, layer_dims=(3 * 32 + 5, 24, 1))
        sup, qry, params = _inputs(cfg, emb_std=0.3)
        if bag > 12:
            off = sup.bag_offsets.clone()
            extra = bag - int(off[1])
            off[1:] += extra
            sup = dataclasses.replace(sup, bag_offsets=off, indices=torch.cat([torch.zeros(extra, dtype=sup.indices.dtype), sup.indices]))
        sets.append((_to_dev(sup, dev), _to_dev(qry, dev)))
    want = None
    for mib in range(400, 90, -12):
        ctx = gm.from_config(cfg, workspace_bytes=mib << 20)
        ctx.configure("row_path", 2)
        p = _params_dev(params, dev)
        with pytest.raises(GMetaError) as e:
            ctx.meta_train(sets, p, cfg.inner_lr, 2, 2, 0.01)
        assert e.value.code == -3 and ctx.iterations_done == 1, f"{mib} MiB: {e.value}"
        ctx.close()
        want = want or p
        assert torch.equal(p.emb, want.emb), f"{mib} MiB"
    assert not torch.equal(want.emb, _params_dev(params, dev).emb)


def test_large_task_whose_matrices_do_not_fit(gm):  # noqa: F811
    """A workspace that holds a large task but not its matrices takes the batch all the same, within rounding."""
    cfg, sup, qry, params = _few_large(12)
    dev = torch.device("cuda", 0)
    s, q, p = _to_dev(sup, dev), _to_dev(qry, dev), _params_dev(params, dev)
    got = []
    for mib in (1024, 160):   # (batch-level buffers and the largest task: 132 MiB, with its 47 MiB of matrices 180)
        ctx = gm.from_config(cfg, workspace_bytes=mib << 20)
        out = ctx.meta_step(s, q, p, cfg.inner_lr, 2, 2)
        got.append(out["emb_grad"][:int(out["n_emb_rows"].item())].clone())
        ctx.close()
    assert not torch.equal(got[0], got[1])   # (the other row arithmetic)
    assert float((got[1] - got[0]).norm()) <= TOL_FP32 * float(got[0].norm())


THREE_STEPS_TOL = 2e-2   # (bf16 operands against float64 on the same gates: up to 5e-3 here)
THREE_STEPS = [(64, [1, 64, 63, 33, 2, 0, 64], [64, 1, 63, 32, 64, 5, 0]), (64, [65, 129, 64, 257, 3, 192], [64, 300, 129, 65, 193, 1]),
               (32, [257, 10, 128, 65], [70, 257, 255, 256])]


def three_steps(D, ns, nq):
    """Inputs that the rows' updates dominate, by about as much in every step: small rows, no dense features (tests/test_oracle_mutations.py
    measures what a step left out does to the results)."""
    F = 3
    cfg = small_cfg(n_tasks=len(ns), n_fields=F, emb_dim=D, rows_per_field=60, n_support=max(ns), n_query=max(nq), bag_max=3, n_dense=0,
                    layer_dims=(F * D, 40, 1), mlp_dtype=1, inner_lr=0.3)
    sup, qry, params = _inputs(cfg, emb_std=0.02)
    return cfg, _cut(sup, ns, F), _cut(qry, nq, F), params


@pytest.mark.parametrize("order", [1, 2])
@pytest.mark.parametrize("D,ns,nq", THREE_STEPS)
def test_sum_of_three_steps(gm, order, D, ns, nq):  # noqa: F811
    """Three inner steps, bf16 operands: the query set's update is one hop of the steps' summed gradients, at the edges of its tiles; with every
    task through the sparse kernel instead, which takes it step by step, the same within the operands' rounding.  Any step left out would
    be three times the tolerance or more."""
    cfg, sup, qry, params = three_steps(D, ns, nq)
    ctx = gm.from_config(cfg, workspace_bytes=1 << 29)
    ctx.configure("row_path", 2)
    a, _ = _compare_step(cfg, ctx, sup, qry, params, 3, order, THREE_STEPS_TOL, f"rows of {D}, {ns} / {nq}", operand="bf16")
    a = [x.clone() for x in (*a["dW"], a["emb_grad"][:int(a["n_emb_rows"].item())])]
    ctx.configure("row_path", 1)
    b = ctx.meta_step(_to_dev(sup, ctx.device), _to_dev(qry, ctx.device), _params_dev(params, ctx.device), cfg.inner_lr, 3, order)
    for x, y in zip(a, (*b["dW"], b["emb_grad"][:int(b["n_emb_rows"].item())])):
        assert float((x - y).norm()) <= THREE_STEPS_TOL * float(y.norm())
    ctx.close()
