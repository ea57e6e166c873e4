"""The kernels that take several arrays in one launch, where their partitions end: scans on both sides of the one-workgroup
limit (16384 values a piece, 32768 in all), pooling with few and with many fields and an odd number of samples, pad rows of
tasks of every remainder modulo the row padding, models with more matrices than one launch takes."""
import numpy as np
import pytest

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


# (the deep model in fp32, at the tighter tolerance: every bf16 layer adds roundings of 2^-9 per operand, and ten layers of them
# reach 2.4e-2 where the tolerance for bf16 is meant for the three or four of the configurations)
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
