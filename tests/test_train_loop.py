"""gm_meta_train: several iterations of Alg. 1 in one call, the index side of batch i+1 prepared on the second stream
while batch i computes.  Through the C ABI: parameters after n iterations equal n calls of gm_meta_train_step bit for
bit (overlapped path and the one-after-the-other fall-back), and follow the oracle's meta_train_step."""
import numpy as np
import pytest
import torch

from oracle import maml_dlrm as O
from synth import SMALL, make_batch, make_params
from synth.generate import Params, SetData
from tests.helpers import oracle_model, rel_err

pytestmark = pytest.mark.gpu


def _clone(p, dev):
    return Params(p.emb.to(dev).clone(), [w.to(dev).clone() for w in p.W], [b.to(dev).clone() for b in p.b])


def _same_params(a, b):
    assert torch.equal(a.emb, b.emb)
    for x, y in zip(a.W + a.b, b.W + b.b):
        assert torch.equal(x, y)


@pytest.mark.parametrize("bf", [0, 1], ids=["fp32", "bf16"])
@pytest.mark.parametrize("mode", ["overlapped", "fallback", "serial"])
def test_train_loop_equals_single_iterations(bf, mode):
    from paper_2401_04338_amd import GMeta
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cfg = SMALL.with_(n_tasks=5, n_support=40, n_query=24, n_fields=6, emb_dim=32, rows_per_field=3000, bag_max=6,
                      layer_dims=(6 * 32 + 13, 64, 32, 1), inner_lr=0.05, mlp_dtype=bf)
    beta, K, order, n = 0.02, 2, 2, 5
    dev = torch.device("cuda", 0)
    params = make_params(cfg, "cpu", emb_std=0.1)
    # batches of different sizes, so that the two index arenas are reused with different layouts
    batches = []
    for it in range(n):
        c_it = cfg.with_(n_tasks=5 - (it % 3))
        s, q = make_batch(c_it, it, dev)
        batches.append((s, q))
    probe = GMeta.from_config(cfg, workspace_bytes=1 << 20)
    need = max(probe.workspace_bytes(len(s.task_offsets) - 1, s.n_samples, q.n_samples, s.nnz, q.nnz, K, order) for s, q in batches)
    probe.close()
    # overlapped: room for two index arenas; fall-back: little more than that; serial: a workspace that holds one batch only
    ws = {"overlapped": 1 << 30, "fallback": int(need * 1.15) + (4 << 20), "serial": need}[mode]
    ctx = GMeta.from_config(cfg, workspace_bytes=ws)
    one = _clone(params, dev)
    want_losses = [float(ctx.meta_train_step(s, q, one, cfg.inner_lr, K, order, beta).item()) for s, q in batches]
    loop = _clone(params, dev)
    ctx.profile(True)
    losses = ctx.meta_train(batches, loop, cfg.inner_lr, K, order, beta)
    ctx.profile(False)
    assert ctx.iterations_done == n
    assert [float(x) for x in losses.cpu()] == want_losses
    _same_params(loop, one)
    # the oracle's training loop on its own copy (fp32 only: the bf16 reference is covered by the single-step tests)
    if not bf:
        ref = params.numpy()
        ref = dict(emb=ref["emb"].astype(np.float64), W=[w.astype(np.float64) for w in ref["W"]], b=[b.astype(np.float64) for b in ref["b"]])
        for (s, q), got in zip(batches, want_losses):
            c_it = cfg.with_(n_tasks=len(s.task_offsets) - 1)
            ref, ref_loss = O.meta_train_step(oracle_model(c_it), ref, s.numpy(), q.numpy(), cfg.inner_lr, K, order, beta)
            assert abs(got - ref_loss) <= 1e-4 * abs(ref_loss)
        moved = max(rel_err(loop.emb.cpu().numpy().astype(np.float64) - params.emb.numpy(), ref["emb"] - params.emb.numpy()))
        assert moved <= 5e-4, moved
    ctx.close()


def test_train_loop_stops_at_a_bad_batch():
    """A batch with an index outside its table in the middle of the loop: the iterations before it are applied (and
    reported), the bad one and the ones after it are not, and the error names the index."""
    from paper_2401_04338_amd import GMeta, GMetaError
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cfg = SMALL.with_(n_tasks=4, n_support=30, n_query=20, n_fields=4, emb_dim=16, rows_per_field=500, bag_max=5,
                      layer_dims=(4 * 16 + 13, 32, 16, 1), inner_lr=0.05)
    dev = torch.device("cuda", 0)
    params = make_params(cfg, "cpu", emb_std=0.1)
    batches = [make_batch(cfg, it, dev) for it in range(4)]
    s, q = batches[2]
    bad = s.indices.clone()
    bad[7] = cfg.rows_per_field
    batches[2] = (SetData(s.task_offsets, s.bag_offsets, bad, s.dense, s.labels), q)
    ctx = GMeta.from_config(cfg, workspace_bytes=1 << 29)
    one, loop = _clone(params, dev), _clone(params, dev)
    for sb, qb in batches[:2]:
        ctx.meta_train_step(sb, qb, one, cfg.inner_lr, 1, 2, 0.05)
    with pytest.raises(GMetaError) as e:
        ctx.meta_train(batches, loop, cfg.inner_lr, 1, 2, 0.05)
    assert e.value.code == -2 and ctx.iterations_done == 2
    _same_params(loop, one)
    # the context keeps working
    ctx.meta_train(batches[:2], loop, cfg.inner_lr, 1, 2, 0.05)
    ctx.close()


def _dense_only_batch(T, n_dense, dev, seed):
    gen = torch.Generator(device=dev).manual_seed(seed)
    toff = np.arange(T + 1, dtype=np.int64)
    none = dict(bag_offsets=torch.zeros(1, dtype=torch.int64, device=dev), indices=torch.zeros(0, dtype=torch.int32, device=dev))
    return tuple(SetData(toff, none["bag_offsets"], none["indices"], torch.randn(T, n_dense, device=dev, generator=gen),
                         (torch.rand(T, device=dev, generator=gen) < 0.5).float()) for _ in range(2))


# a batch of more tasks than a wave may hold (65535: the most blocks in a grid's y), and one cut by "max_wave_tasks"
@pytest.mark.parametrize("tasks,per_wave", [(65536, 0), (32769, 0), (300, 128)])
def test_train_loop_with_more_tasks_than_a_wave(tasks, per_wave):
    from paper_2401_04338_amd import GMeta
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda", 0)
    dims = [5, 4, 1]
    gen = torch.Generator(device=dev).manual_seed(1)
    params = Params(torch.zeros(0, 4, device=dev), [torch.randn(a, b, device=dev, generator=gen) for a, b in zip(dims[:-1], dims[1:])],
                    [torch.randn(b, device=dev, generator=gen) for b in dims[1:]])
    batches = [_dense_only_batch(tasks, 5, dev, 7 + i) for i in range(2)]
    ctx = GMeta(0, [], 4, 5, dims, 0, workspace_bytes=6 << 30)   # (holds the loop's two batches as one wave each)
    ctx.configure("max_wave_tasks", per_wave)
    one, loop = _clone(params, dev), _clone(params, dev)
    want = [float(ctx.meta_train_step(s, q, one, 0.05, 1, 2, 1e-4).item()) for s, q in batches]
    losses = ctx.meta_train(batches, loop, 0.05, 1, 2, 1e-4)
    assert ctx.iterations_done == 2 and [float(x) for x in losses.cpu()] == want
    _same_params(loop, one)
    assert all(torch.isfinite(w).all() for w in loop.W)
    ctx.close()


@pytest.mark.parametrize("dim,rows,bf", [(4, 3, 0), (32, 700, 0), (64, 5, 1), (256, 40, 0)])
@pytest.mark.parametrize("waves", [1, 2])
def test_update_of_the_rows_inside_the_step(dim, rows, bf, waves):
    """One wave of tasks: the segment reduction adds to the tables itself.  The parameters are those of the step's list applied
    by gm_scatter_add, bit for bit; several waves take the list, or the caller's table-shaped buffer, as before."""
    from paper_2401_04338_amd import GMeta
    cfg = SMALL.with_(n_tasks=12, n_support=50, n_query=40, n_fields=3, emb_dim=dim, rows_per_field=rows, bag_max=9,
                      layer_dims=(3 * dim + 13, 32, 1), inner_lr=0.05, mlp_dtype=bf)
    beta, K, order, dev = 0.02, 1, 2, torch.device("cuda", 0)
    params = make_params(cfg, "cpu", emb_std=0.1)
    s, q = make_batch(cfg, 0, dev)
    ctx = GMeta.from_config(cfg, workspace_bytes=1 << 30)
    ctx.configure("max_wave_tasks", -(-cfg.n_tasks // waves))
    want = _clone(params, dev)
    out = ctx.meta_step(s, q, want, cfg.inner_lr, K, order)
    n = int(out["n_emb_rows"].item())
    ctx.scatter_add(want.emb, out["emb_rows"][:n].contiguous(), out["emb_grad"][:n].contiguous(), -beta)
    got = _clone(params, dev)
    loss = ctx.meta_train_step(s, q, got, cfg.inner_lr, K, order, beta)
    assert float(loss.item()) == float(out["loss"].item())
    assert torch.equal(got.emb, want.emb)
    by_table, table = _clone(params, dev), torch.zeros(3 * rows, dim, device=dev)
    ctx.meta_train_step_table(s, q, by_table, cfg.inner_lr, K, order, beta, table)
    assert not table.any()
    if waves == 1:
        _same_params(by_table, got)
    else:      # (two sums per row, added: fp32 rounding of at most three additions more)
        moved = (want.emb - params.emb.to(dev)).abs().max()
        assert (by_table.emb - got.emb).abs().max() <= 1e-5 * moved + 2 * torch.finfo(torch.float32).eps * want.emb.abs().max()
    ctx.close()


def test_workspace_without_room_for_the_lists():
    """Many distinct rows: the row lists take more than a batch's index structures, so between the sizes at which the loop overlaps and at
    which the lists fit beside one wave, single iterations have to run as one wave without lists to give the loop's bits (40 tasks:
    other waves would sum the hidden layers' gradients over other runs of tasks)."""
    from paper_2401_04338_amd import GMeta
    cfg = SMALL.with_(n_tasks=40, n_support=30, n_query=30, n_fields=6, emb_dim=64, rows_per_field=30000, bag_max=20, zipf_s=0.0,
                      layer_dims=(6 * 64 + 13, 32, 1), inner_lr=0.05)
    beta, K, order, dev = 0.02, 1, 2, torch.device("cuda", 0)
    params = make_params(cfg, "cpu", emb_std=0.1)
    batches = [make_batch(cfg, it, dev) for it in range(2)]
    s, q = batches[0]
    probe = GMeta.from_config(cfg, workspace_bytes=1 << 20)
    need = probe.workspace_bytes(cfg.n_tasks, s.n_samples, q.n_samples, s.nnz, q.nnz, K, order)
    probe.close()
    lists = min(s.nnz + q.nnz, 6 * 30000) * (4 * 64 + 8)
    for extra in range(12):   # from one wave to room for the loop's two batches and the lists
        ctx = GMeta.from_config(cfg, workspace_bytes=need + extra * lists // 6)
        one, loop = _clone(params, dev), _clone(params, dev)
        ctx.profile(True)
        for sb, qb in batches:
            ctx.meta_train_step(sb, qb, one, cfg.inner_lr, K, order, beta)
        assert "scatter_add" not in ctx.profile_report()   # (no list applied: one wave)
        ctx.profile(False)
        ctx.meta_train(batches, loop, cfg.inner_lr, K, order, beta)
        ctx.close()
        _same_params(loop, one)
