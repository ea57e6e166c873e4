"""The fp32 products at the edges of their tiles: task sizes around 32 and 64 rows, widths that are not multiples of 32
or 64, contractions that end inside a piece, and batches on either side of the rule that picks the tile shape
(the last one's first layer has 600 tiles of 64 x 64)."""
import pytest
import torch

from tests.helpers import small_cfg
from tests.test_gpu_parity import TOL_FP32, _compare_step, _inputs, _params_dev, _to_dev, gm  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tasks,rows,hidden", [(1, 1, (1,)), (2, 31, (33, 5)), (3, 65, (64, 32)), (5, 130, (129, 63, 31)),
                                               (100, 20, (330,))])
def test_tile_edges(gm, tasks, rows, hidden):  # noqa: F811
    cfg = small_cfg(n_tasks=tasks, n_support=rows, n_query=max(1, rows - 1), layer_dims=(17,) + hidden + (1,))
    sup, qry, params = _inputs(cfg, emb_std=0.3)
    ctx = gm.from_config(cfg, workspace_bytes=1 << 28)
    _compare_step(cfg, ctx, sup, qry, params, 2, 2, TOL_FP32, f"{tasks} tasks x {rows}, {hidden}")
    ctx.close()


@pytest.mark.parametrize("tasks,hidden,waves", [(100, (330, 70), (50, 9)),    # 600 tiles in the first layer: 300 and 54 in a wave
                                                (40, (129, 31), (39, 7))])   # few tiles, and a wave of one task at the end
@pytest.mark.parametrize("order", [1, 2])
def test_bits_do_not_depend_on_the_wave(gm, tasks, hidden, waves, order):  # noqa: F811
    """A task's loss and its share of the sparse gradient have the same bits whatever shares its launches."""
    cfg = small_cfg(n_tasks=tasks, n_support=20, n_query=19, layer_dims=(17,) + hidden + (1,))
    sup, qry, params = _inputs(cfg, emb_std=0.3)
    ctx = gm.from_config(cfg, workspace_bytes=1 << 28)
    dev = ctx.device
    s, q, p = _to_dev(sup, dev), _to_dev(qry, dev), _params_dev(params, dev)
    ref = ctx.meta_step(s, q, p, cfg.inner_lr, 2, order)
    n = int(ref["n_emb_rows"].item())
    for per in waves:
        ctx.configure("max_wave_tasks", per)
        got = ctx.meta_step(s, q, p, cfg.inner_lr, 2, order)
        assert torch.equal(got["task_loss"][:tasks], ref["task_loss"][:tasks]), per
        assert int(got["n_emb_rows"].item()) == n and torch.equal(got["emb_rows"][:n], ref["emb_rows"][:n]), per
        assert torch.equal(got["emb_grad"][:n], ref["emb_grad"][:n]), per
        for a, b in zip(got["dW"] + got["db"], ref["dW"] + ref["db"]):   # (summed over other runs of tasks)
            assert float((a - b).abs().max()) <= 1e-5 * float(b.abs().max()) + 1e-9, per
    ctx.close()
