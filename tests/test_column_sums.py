"""The per-task column sums: more sums than one launch takes, rows that end inside a wave's batch, widths of several
column blocks and widths that leave lanes of a row group empty, tasks with rows for some of the waves only."""
import pytest

from tests.helpers import small_cfg
from tests.test_gpu_parity import TOL_FP32, _compare_step, _inputs, gm  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf,tasks,rows,hidden", [(0, 2, 3, (12,) * 13), (0, 3, 129, (300, 40)), (0, 2, 513, (9,)),
                                                  (1, 3, 65, (600, 72)), (1, 2, 133, (40,)),
                                                  (0, 5, 8, (300, 40)), (0, 5, 16, (300, 40)), (1, 5, 4, (600, 72)), (1, 5, 31, (600, 72))])
def test_partitions(gm, bf, tasks, rows, hidden):  # noqa: F811
    cfg = small_cfg(n_tasks=tasks, n_support=rows, n_query=max(1, rows - 2), layer_dims=(17,) + hidden + (1,), mlp_dtype=bf)
    sup, qry, params = _inputs(cfg, emb_std=0.3)
    ctx = gm.from_config(cfg, workspace_bytes=1 << 28)
    _compare_step(cfg, ctx, sup, qry, params, 2, 2, 2e-2 if bf else TOL_FP32, f"{tasks} x {rows}, {hidden}", operand="bf16" if bf else "fp64")
    ctx.close()
