"""The kernels that take several arrays in one launch, where their partitions end: scans on both sides of the one-workgroup
limit (16384 values a piece, 32768 in all), pooling with few and with many fields and an odd number of samples, pad rows of
tasks of every remainder modulo the row padding, models with more matrices than one launch takes."""
from types import SimpleNamespace

import numpy as np
import pytest
import torch

from oracle import maml_dlrm as O
from tests.helpers import oracle_model, small_cfg
from tests.test_gpu_parity import TOL_FP32, _compare_step, _inputs, _to_dev, gm  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tasks", [2047, 2048, 2049, 4096, 4097])   # x 8 (task, field) counts
def test_scan_lengths(gm, tasks):  # noqa: F811
    cfg = small_cfg(n_tasks=tasks, n_fields=8, n_support=2, n_query=1, rows_per_field=300, bag_max=2)
    sup, qry, _ = _inputs(cfg)
    ctx = gm.from_config(cfg, workspace_bytes=1 << 28)
    got = ctx.index_prep(_to_dev(sup, ctx.device), _to_dev(qry, ctx.device))
    ref = O.index_prep(oracle_model(cfg), sup.numpy(), qry.numpy())
    for k in ("slot_counts", "slot_rows", "sup_slot", "qry_slot", "emb_rows", "seg_counts"):
        assert np.array_equal(got[k].cpu().numpy(), ref[k]), k
    ctx.close()


# (the deep model in fp32: every bf16 layer adds roundings of 2^-9 per operand, and ten layers of random weights reach 2.4e-2
# where the tolerance for bf16 is meant for the three or four of the configurations; its bf16 packing is compared below)
# (fields, rows): below eight fields / below 16384 bags one kernel pools, from there on the one that deals fields to the XCDs
@pytest.mark.parametrize("bf,fields,tasks,rows,hidden", [(0, 3, 3, 33, (8, 6)), (0, 9, 7, 131, (40,)), (0, 8, 4, 256, (8,)),
                                                         (1, 9, 9, 133, (40, 24)), (0, 11, 2, 9, (16,) * 9)])
def test_both_sets_in_one_launch(gm, bf, fields, tasks, rows, hidden):  # noqa: F811
    d0 = fields * 16 + 5
    cfg = small_cfg(n_tasks=tasks, n_fields=fields, emb_dim=16, n_support=rows, n_query=rows - 2 if rows % 2 else rows, layer_dims=(d0,) + hidden + (1,),
                    mlp_dtype=bf)
    sup, qry, params = _inputs(cfg, emb_std=0.3)
    ctx = gm.from_config(cfg, workspace_bytes=1 << 29)
    for order in (1, 2):
        _compare_step(cfg, ctx, sup, qry, params, 2, order, 2e-2 if bf else TOL_FP32, f"{fields} fields, {tasks} x {rows}",
                      operand="bf16" if bf else "fp64")
    ctx.close()


# ten layers: twenty matrices, more than one launch packs.  Hidden weights are permutations and inputs and biases small whole
# numbers, so that every activation is a whole number below 2^8 and exact in bf16 as in fp32: only the last product and the loss round.
@pytest.mark.parametrize("bf", [0, 1])
def test_weights_of_many_layers(gm, bf):  # noqa: F811
    rng = np.random.default_rng(5)
    D, width, layers, tasks, rows = 4, 32, 9, 3, 9
    dims = [D + width] + [width] * layers + [1]
    perms = [rng.permutation(width) for _ in range(layers)]
    W = [np.zeros((a, b), dtype=np.float32) for a, b in zip(dims[:-1], dims[1:])]
    for l, p in enumerate(perms):
        W[l][(D if l == 0 else 0) + p, np.arange(width)] = 1.0
    W[-1][:, 0] = rng.standard_normal(width) / 64
    b = [rng.integers(0, 4, n).astype(np.float32) for n in dims[1:-1]] + [np.full(1, 0.25, np.float32)]
    x, y = rng.integers(0, 8, (tasks * rows, width)).astype(np.float32), (rng.random(tasks * rows) < 0.5).astype(np.float32)
    a = x.astype(np.float64)
    for p, c in zip(perms, b):
        a = a[:, p] + c
    assert a.max() < 256
    z = a @ W[-1].astype(np.float64)[:, 0] + 0.25
    want = (np.maximum(z, 0) - y * z + np.log1p(np.exp(-np.abs(z)))).reshape(tasks, rows).mean(1)
    dev = "cuda:0"
    batch = SimpleNamespace(task_offsets=np.arange(tasks + 1, dtype=np.int64) * rows, labels=torch.from_numpy(y).to(dev), dense=torch.from_numpy(x).to(dev),
                            bag_offsets=torch.zeros(tasks * rows + 1, dtype=torch.int64, device=dev), indices=torch.zeros(0, dtype=torch.int32, device=dev))
    params = SimpleNamespace(emb=torch.zeros(3, D, device=dev), W=[torch.from_numpy(w).to(dev) for w in W], b=[torch.from_numpy(c).to(dev) for c in b])
    ctx = gm(1, [3], D, width, dims, bf, workspace_bytes=1 << 26)
    out = ctx.meta_step(batch, batch, params, 0.1, 0, 1)
    # 33 fp32 products and sums of the logit, and the exponential and the logarithm to a few units in the last place
    scale = float(np.abs(a * W[-1][:, 0]).sum(1).max())
    assert np.max(np.abs(out["task_loss"][:tasks].cpu().numpy() - want)) <= 40 * 2.0 ** -24 * scale
    # the gradient of every bias comes back too: the row's delta times the last weights, carried back through the permutations (in
    # bf16 rounded once, then moved whole), summed over the rows and tasks in fp32
    delta = (1 / (1 + np.exp(-z)) - y) / rows
    g = delta[:, None] * W[-1].astype(np.float64)[:, 0] * (a > 0)
    act = a
    for l in range(layers - 1, -1, -1):
        tol = (2.0 ** -8 if bf else 2.0 ** -20) * np.abs(g).sum(0) + tasks * 2.0 ** -21 * np.abs(W[-1]).max()   # (the sigmoid to 8 units of 2^-24)
        assert np.all(np.abs(out["db"][l].cpu().numpy() - g.sum(0)) <= tol), l
        act = act - b[l]
        g = g[:, np.argsort(perms[l])]
        act = act[:, np.argsort(perms[l])]
        g = g * (act > 0)
    ctx.close()
