"""The fp32 products at the edges of their tiles: task sizes around 32 and 64 rows, widths that are not multiples of 32
or 64, contractions that end inside a piece, and batches on either side of the rule that picks the tile shape
(the last one's first layer has 600 tiles of 64 x 64)."""
import pytest

from tests.helpers import small_cfg
from tests.test_gpu_parity import TOL_FP32, _compare_step, _inputs, gm  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tasks,rows,hidden", [(1, 1, (1,)), (2, 31, (33, 5)), (3, 65, (64, 32)), (5, 130, (129, 63, 31)),
                                               (100, 20, (330,))])
def test_tile_edges(gm, tasks, rows, hidden):  # noqa: F811
    cfg = small_cfg(n_tasks=tasks, n_support=rows, n_query=max(1, rows - 1), layer_dims=(17,) + hidden + (1,))
    sup, qry, params = _inputs(cfg, emb_std=0.3)
    ctx = gm.from_config(cfg, workspace_bytes=1 << 28)
    _compare_step(cfg, ctx, sup, qry, params, 2, 2, TOL_FP32, f"{tasks} tasks x {rows}, {hidden}")
    ctx.close()
