"""Second-order steps of small tasks whose direction on the hidden layers' weights stays factors (gm_configure "chain_factors"): against the oracle,
with tasks of one row, of a tile's edges, without support or query rows, of more rows in one set than the other, one to four
inner steps, one and several hidden layers, rows adapted or not, one wave and several."""
import pytest

from synth import SMALL
from tests.helpers import small_cfg
from tests.test_gpu_parity import TOL_BF16, _compare_step, _inputs, gm  # noqa: F401
from tests.test_hop_tiles import _cut

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ns,nq,hidden,K,adapt", [
    ([30, 8, 64, 1, 65, 17], [30, 64, 8, 20, 17, 1], (64,), 1, 1),
    ([24, 33, 2, 9, 40, 16], [31, 7, 12, 40, 9, 16], (136, 40), 2, 1),
    ([24, 33, 2, 9, 40, 16], [31, 7, 12, 40, 9, 16], (136, 40), 2, 0),
    ([70, 5, 129, 12], [6, 90, 40, 130], (96, 64, 32), 2, 1),
    ([20, 31, 12], [25, 9, 16], (72, 40), 3, 1),
    ([20, 12], [9, 16], (64, 32), 4, 1),
    ([20, 8, 12], [0, 9, 16], (64, 32), 2, 1)])
def test_factors_against_the_oracle(gm, ns, nq, hidden, K, adapt):  # noqa: F811
    F, D = 5, 32
    cfg = SMALL.with_(n_tasks=len(ns), n_support=max(ns), n_query=max(nq), n_fields=F, emb_dim=D, rows_per_field=300, bag_max=5,
                      layer_dims=(F * D + 13, *hidden, 1), inner_lr=0.05, mlp_dtype=1)
    sup, qry, params = _inputs(cfg, emb_std=0.2)
    sup, qry = _cut(sup, ns, F), _cut(qry, nq, F)
    ctx = gm.from_config(cfg, workspace_bytes=1 << 30)
    ctx.configure("chain_factors", 2)
    ctx.configure("adapt_rows", adapt)
    _compare_step(cfg, ctx, sup, qry, params, K, 2, TOL_BF16, f"{ns} / {nq} rows, {hidden}, K={K}", operand="bf16", adapt_rows=bool(adapt))
    ctx.close()
