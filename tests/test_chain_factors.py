"""Second-order steps of small tasks whose direction on the hidden layers' weights stays factors (gm_configure "chain_factors"): against the oracle
and, the second-order part by itself, against the matrices, with tasks of one row, of a tile's edges, without support or query rows, of
more rows in one set than the other, one to four inner steps, one and several hidden layers, rows adapted or not, one wave and
several; and that the rule by sizes takes factors."""
import pytest
import torch

from synth import SMALL
from tests.helpers import small_cfg
from tests.test_gpu_parity import TOL_BF16, _compare_step, _inputs, _params_dev, _to_dev, gm  # noqa: F401
from tests.test_hop_tiles import _cut

pytestmark = pytest.mark.gpu

SHAPES = pytest.mark.parametrize("ns,nq,hidden,K,adapt", [
    ([30, 8, 64, 1, 65, 17], [30, 64, 8, 20, 17, 1], (64,), 1, 1),
    ([24, 33, 2, 9, 40, 16], [31, 7, 12, 40, 9, 16], (136, 40), 2, 1),
    ([24, 33, 2, 9, 40, 16], [31, 7, 12, 40, 9, 16], (136, 40), 2, 0),
    ([70, 5, 129, 12], [6, 90, 40, 130], (96, 64, 32), 2, 1),
    ([20, 31, 12], [25, 9, 16], (72, 40), 3, 1),
    ([20, 12], [9, 16], (64, 32), 4, 1),
    ([20, 8, 12], [0, 9, 16], (64, 32), 2, 1)])


def _batch(ns, nq, hidden, F=5, D=32):
    cfg = SMALL.with_(n_tasks=len(ns), n_support=max(ns), n_query=max(nq), n_fields=F, emb_dim=D, rows_per_field=300, bag_max=5,
                      layer_dims=(F * D + 13, *hidden, 1), inner_lr=0.05, mlp_dtype=1)
    sup, qry, params = _inputs(cfg, emb_std=0.2)
    return cfg, _cut(sup, ns, F), _cut(qry, nq, F), params


@SHAPES
def test_factors_against_the_oracle(gm, ns, nq, hidden, K, adapt):  # noqa: F811
    cfg, sup, qry, params = _batch(ns, nq, hidden)
    ctx = gm.from_config(cfg, workspace_bytes=1 << 30)
    ctx.configure("chain_factors", 2)
    ctx.configure("adapt_rows", adapt)
    _compare_step(cfg, ctx, sup, qry, params, K, 2, TOL_BF16, f"{ns} / {nq} rows, {hidden}, K={K}", operand="bf16", adapt_rows=bool(adapt))
    ctx.close()


def _outputs(ctx, s, q, p, cfg, K, order, factors, wave):
    ctx.configure("chain_factors", factors)
    ctx.configure("max_wave_tasks", wave)
    out = ctx.meta_step(s, q, p, cfg.inner_lr, K, order)
    return out["task_loss"][:cfg.n_tasks].clone(), out["emb_grad"][:int(out["n_emb_rows"].item())].clone(), [w.clone() for w in out["dW"]]


@SHAPES
@pytest.mark.parametrize("wave", [0, 2])
def test_factors_against_matrices(gm, ns, nq, hidden, K, adapt, wave):  # noqa: F811
    """The second-order part of the meta-gradient (what it differs by from the first order's, same adapted weights) with factors and with
    matrices, whose only difference is that a matrix is rounded to bf16: a factor's missing or doubled tile would be a large
    part of it.  A wave's borders change no bit of losses and row gradients."""
    cfg, sup, qry, params = _batch(ns, nq, hidden)
    ctx = gm.from_config(cfg, workspace_bytes=1 << 30)
    ctx.configure("adapt_rows", adapt)
    ctx.configure("theta_from_meta", 0)   # (the adapted weights then are the same bits in either order)
    args = ctx, _to_dev(sup, ctx.device), _to_dev(qry, ctx.device), _params_dev(params, ctx.device), cfg, K
    first, matrices, factors = (_outputs(*args, order, way, wave) for order, way in ((1, 0), (2, 1), (2, 2)))
    assert torch.equal(first[0], matrices[0]) and torch.equal(factors[0], matrices[0])
    for a, m, f in zip([first[1], *first[2][:-1]], [matrices[1], *matrices[2][:-1]], [factors[1], *factors[2][:-1]]):
        part = (m - a).double()
        assert float((f - m).double().norm()) <= 2 ** -8 * float(part.norm())   # (bf16 rounds by at most 2^-9 of a value)
        assert not torch.equal(f, m)      # (factors are what ran)
    if wave:
        whole = _outputs(*args, 2, 2, 0)
        assert torch.equal(whole[0], factors[0]) and torch.equal(whole[1], factors[1])
        for a, b in zip(whole[2], factors[2]):
            assert float((a - b).norm()) <= 1e-6 * float(a.norm())
    ctx.close()


@pytest.mark.parametrize("wave", [0, 40])
def test_rule_by_sizes(gm, wave):  # noqa: F811
    """Many small tasks under layers wide enough that their matrices would not stay in the memory-side cache: factors by default."""
    ns, nq = [16, 9, 24] * 32, [8, 30, 11] * 32
    cfg, sup, qry, params = _batch(ns, nq, (512, 32), F=31)
    ctx = gm.from_config(cfg, workspace_bytes=4 << 30)
    args = ctx, _to_dev(sup, ctx.device), _to_dev(qry, ctx.device), _params_dev(params, ctx.device), cfg, 2, 2
    default, matrices, factors = (_outputs(*args, way, wave) for way in (0, 1, 2))
    ctx.close()
    for i in range(2):
        assert torch.equal(default[i], factors[i])
    assert not torch.equal(default[1], matrices[1])
    assert all(torch.equal(a, b) for a, b in zip(default[2], factors[2]))
