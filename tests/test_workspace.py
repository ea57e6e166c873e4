"""Workspace that calls need: no more than they used to, with the same results in any."""
import pytest
import torch

from paper_2401_04338_amd.binding import _model_desc, load_library

BAG, ROWS, N_DENSE = 5, 100_000, 13
# (fields, columns, hidden layers, tasks, support and query samples a task, bf16, order): bytes for 0..5 inner steps as commit 5cad85f asked for
FORMER = {
    (26, 64, '512-256', 201, 150, 243, 0, 1): [3350248960, 4597006080, 4994194944, 4994194944, 4994194944, 4994194944],
    (26, 64, '512-256', 201, 150, 243, 0, 2): [3350248960, 5243774464, 6630832640, 7825239552, 9019646464, 10214053376],
    (26, 64, '128-64', 201, 340, 243, 0, 1): [3352852992, 4153484800, 5387708416, 5387708416, 5387708416, 5387708416],
    (26, 64, '128-64', 201, 340, 243, 0, 2): [3352852992, 5236083712, 6757181184, 7507673600, 8258166016, 9008658432],
    (64, 64, '1024-512-256', 128, 512, 512, 0, 1): [12176156160, 17764595968, 20994210048, 20994210048, 20994210048, 20994210048],
    (64, 64, '1024-512-256', 128, 512, 512, 0, 2): [12176156160, 21933996544, 28604529664, 33127579136, 37650628608, 42173678080],
    (64, 64, '1024-512-256', 48, 9, 9, 0, 1): [1353192960, 2309801216, 2329517312, 2329517312, 2329517312, 2329517312],
    (64, 64, '1024-512-256', 48, 9, 9, 0, 2): [1353192960, 2335712256, 3299451392, 4250607616, 5201763840, 6152920064],
    (8, 16, '64-32', 4, 32, 32, 0, 1): [3160320, 3459328, 3541248, 3541248, 3541248, 3541248],
    (8, 16, '64-32', 4, 32, 32, 0, 2): [3160320, 3640320, 4021248, 4402176, 4783104, 5164032],
    (11, 32, '100-52', 37, 45, 61, 0, 1): [44942080, 57712384, 61936896, 61936896, 61936896, 61936896],
    (11, 32, '100-52', 37, 45, 61, 0, 2): [44942080, 64501248, 79826688, 93485056, 107143424, 120801792],
    (26, 64, '', 20, 64, 64, 0, 1): [69350912, 71631104, 82444544, 82444544, 82444544, 82444544],
    (26, 64, '', 20, 64, 64, 0, 2): [69350912, 82449920, 93412352, 102244864, 111077376, 119909888],
    (4, 64, '2048-1024', 300, 200, 20, 0, 1): [3853890304, 8577930240, 8725693440, 8725693440, 8725693440, 8725693440],
    (4, 64, '2048-1024', 300, 200, 20, 0, 2): [3853890304, 10141511168, 14993639424, 19767124480, 24540609536, 29314094592],
    (26, 64, '512-256', 700, 52, 52, 0, 1): [5079464192, 8179308544, 8500793344, 8500793344, 8500793344, 8500793344],
    (26, 64, '512-256', 700, 52, 52, 0, 2): [5079464192, 8724580608, 12071342336, 15343556864, 18615771392, 21887985920],
    (26, 32, '256-128', 1, 8, 2, 0, 1): [20631552, 21782528, 21916672, 21916672, 21916672, 21916672],
    (26, 32, '256-128', 1, 8, 2, 0, 2): [20631552, 21941504, 23118848, 24189696, 25260544, 26331392],
    (26, 64, '512-256', 201, 150, 243, 1, 2): [3494604288, 5836948480, 6635812608, 7242025472, 7848238336, 8454451200],
    (26, 64, '128-64', 201, 340, 243, 1, 2): [3293747200, 5647458816, 6799384320, 7180704768, 7562025216, 7943345664],
    (64, 64, '1024-512-256', 128, 512, 512, 1, 2): [12512465664, 23705263872, 28127962112, 30403176704, 32678391296, 34953605888],
    (64, 64, '1024-512-256', 48, 9, 9, 1, 2): [1857811200, 3325905152, 3819104768, 4299721472, 4780338176, 5260954880],
    (8, 16, '64-32', 4, 32, 32, 1, 2): [3292928, 3914752, 4126208, 4337664, 4549120, 4760576],
    (11, 32, '100-52', 37, 45, 61, 1, 2): [48127488, 73129216, 82021632, 89246976, 96472320, 103697664],
    (26, 64, '', 20, 64, 64, 1, 2): [70183424, 93868800, 100964352, 105929984, 110895616, 115861248],
    (4, 64, '2048-1024', 300, 200, 20, 1, 2): [5432613376, 11983455744, 14474866176, 16887633408, 19300400640, 21713167872],
    (26, 64, '512-256', 700, 52, 52, 1, 2): [6441468928, 11605725440, 13347478272, 15014683904, 16681889536, 18349095168],
    (26, 32, '256-128', 1, 8, 2, 1, 2): [21783296, 23676672, 24342272, 24901376, 25460480, 26019584],
    (26, 64, '512-256', 201, 150, 243, 1, 1): [3494604288, 5161885184, 5461577984, 5461577984, 5461577984, 5461577984],
    (26, 64, '128-64', 201, 340, 243, 1, 1): [3293747200, 4370130944, 5377317888, 5377317888, 5377317888, 5377317888],
    (64, 64, '1024-512-256', 128, 512, 512, 1, 1): [12512465664, 19435940096, 22131886592, 22131886592, 22131886592, 22131886592],
    (64, 64, '1024-512-256', 48, 9, 9, 1, 1): [1857811200, 3288790272, 3307714048, 3307714048, 3307714048, 3307714048],
    (8, 16, '64-32', 4, 32, 32, 1, 1): [3292928, 3703040, 3753216, 3753216, 3753216, 3753216],
    (11, 32, '100-52', 37, 45, 61, 1, 1): [48127488, 65542400, 68687360, 68687360, 68687360, 68687360],
    (26, 64, '', 20, 64, 64, 1, 1): [70183424, 77282816, 84229632, 84229632, 84229632, 84229632],
    (4, 64, '2048-1024', 300, 200, 20, 1, 1): [5432613376, 11093151488, 11207564544, 11207564544, 11207564544, 11207564544],
    (26, 64, '512-256', 700, 52, 52, 1, 1): [6441468928, 10983869184, 11198506240, 11198506240, 11198506240, 11198506240],
    (26, 32, '256-128', 1, 8, 2, 1, 1): [21783296, 23467776, 23600384, 23600384, 23600384, 23600384],
}


@pytest.mark.parametrize("shape", FORMER, ids=lambda s: "-".join(str(x) for x in s))
def test_no_more_than_it_was(shape):
    import ctypes as C
    F, D, hidden, T, S, Q, bf16, order = shape
    dims = [F * D + N_DENSE] + [int(h) for h in hidden.split("-") if h] + [1]
    desc = _model_desc(F, [ROWS] * F, D, N_DENSE, dims, bf16)
    for K, most in enumerate(FORMER[shape]):
        need = load_library().gm_workspace_bytes(C.byref(desc), T, T * S, T * Q, T * S * F * BAG, T * Q * F * BAG, K, order)
        assert 0 < need <= most, (K, need - most)


# What a call needs in KiB, with steps of 16, as commit 5cad85f needed it: gm_meta_train_step, gm_meta_step as one wave of tasks
FORMER_KIB = {((128, 64), 3, 128, 128): (115008, 116208), ((128, 64), 3, 160, 40): (109712, 110560), ((128, 64), 2, 128, 128): (115008, 116208),
              ((512, 256), 3, 128, 128): (174368, 264896), ((512, 256), 3, 160, 40): (145888, 256224), ((512, 256), 2, 128, 128): (174368, 264896)}


def _first_order(hidden, n_support, n_query, **kw):
    from synth import SMALL
    from tests.test_gpu_parity import _inputs, _params_dev, _to_dev
    cfg = SMALL.with_(n_tasks=24, n_support=n_support, n_query=n_query, n_fields=10, emb_dim=64, rows_per_field=60000, bag_max=12,
                      layer_dims=(10 * 64 + N_DENSE,) + hidden + (1,), mlp_dtype=1, inner_lr=0.05, **kw)
    sup, qry, params = _inputs(cfg)
    dev = torch.device("cuda", 0)
    return cfg, _to_dev(sup, dev), _to_dev(qry, dev), _params_dev(params, dev)


def _waves(ctx):
    return ctx.profile_report()["gather_pool"]["launches"]


def _step(ctx, cfg, s, q, p, K, order=1):
    out = ctx.meta_step(s, q, p, cfg.inner_lr, K, order)
    n = int(out["n_emb_rows"].item())
    return [out["loss"], out["emb_rows"][:n], out["emb_grad"][:n]] + out["dW"] + out["db"]


@pytest.mark.gpu
@pytest.mark.parametrize("shape", FORMER_KIB, ids=str)
def test_first_order_in_the_former_workspace(shape):
    """One wave of tasks, and training steps, in what they needed before a first-order call's steps kept anything: the same bits as with room to spare."""
    from paper_2401_04338_amd import GMeta
    hidden, K, n_support, n_query = shape
    cfg, s, q, p = _first_order(hidden, n_support, n_query)
    train_kib, wave_kib = FORMER_KIB[shape]
    steps = []
    for kib in (wave_kib, 2 << 20):
        ctx = GMeta.from_config(cfg, workspace_bytes=kib << 10)
        ctx.profile(True)
        steps.append(_step(ctx, cfg, s, q, p, K))
        assert _waves(ctx) == 1
        ctx.close()
    assert all(torch.equal(x, y) for x, y in zip(*steps))
    for kib in (train_kib, 2 << 20):
        ctx = GMeta.from_config(cfg, workspace_bytes=kib << 10)
        for run in (lambda: ctx.meta_train_step(s, q, p, cfg.inner_lr, K, 1, 0.0), lambda: ctx.meta_train([(s, q), (s, q)], p, cfg.inner_lr, K, 1, 0.0)):
            loss = run()   # (outer learning rate 0: the parameters stay)
            assert torch.allclose(loss, steps[0][0].expand_as(loss), rtol=1e-3)
        ctx.close()


@pytest.mark.gpu
def test_first_order_in_waves():
    """Uneven tasks in less and less workspace: no more waves of tasks than without the steps' activations, and no other results than
    rounding makes."""
    from paper_2401_04338_amd import GMeta
    cfg, s, q, p = _first_order((128, 64), 0, 0, lognormal_sizes=True, size_median=60, size_sigma=1.0, size_max=500)
    whole = None
    seen = set()
    for share in (1.0, 0.6, 0.45, 0.35, 0.28, 0.2):
        waves = []
        for from_meta in (1, 0):
            probe = GMeta.from_config(cfg, workspace_bytes=1 << 20)
            need = probe.workspace_bytes(24, s.n_samples, q.n_samples, s.nnz, q.nnz, 3, 1)
            probe.close()
            ctx = GMeta.from_config(cfg, workspace_bytes=int(1.2 * need * share))
            ctx.configure("theta_from_meta", from_meta)
            ctx.profile(True)
            got = _step(ctx, cfg, s, q, p, 3)
            waves.append(_waves(ctx))
            ctx.close()
            whole = whole or got
            assert torch.equal(got[1], whole[1])
            for x, y in zip(got[2:], whole[2:]):
                assert float((x - y).norm()) <= 5e-3 * float(y.norm()), (share, from_meta)
        assert waves[0] <= waves[1]
        seen.add(waves[0])
    assert len(seen) >= 3, seen


@pytest.mark.gpu
@pytest.mark.parametrize("n_support,n_query", [(40, 56), (56, 40), (130, 20)])
@pytest.mark.parametrize("table", [False, True])
def test_first_order_whatever_the_workspace_held(n_support, n_query, table):
    """Steps' activations and gradients lie in memory that the outer pass then uses: the same bits in a fresh context, and after calls of
    other kinds in the same one."""
    from paper_2401_04338_amd import GMeta
    cfg, s, q, p = _first_order((256, 64), n_support, n_query)

    def step(ctx, K, order):
        if not table:
            return _step(ctx, cfg, s, q, p, K, order)
        sums = torch.zeros_like(p.emb)
        out = ctx.meta_step(s, q, p, cfg.inner_lr, K, order, emb_grad_table=sums)
        return [out["loss"], sums] + out["dW"] + out["db"]
    used = GMeta.from_config(cfg, workspace_bytes=1 << 30)
    for K in (2, 3, 4):
        fresh = GMeta.from_config(cfg, workspace_bytes=1 << 30)
        want = step(fresh, K, 1)
        fresh.close()
        step(used, K, 2)
        assert all(torch.equal(x, y) for x, y in zip(step(used, K, 1), want)), K
    used.close()


@pytest.mark.gpu
@pytest.mark.parametrize("rows,from_meta", [(396, True), (408, False)])
def test_first_order_weights_on_both_sides_of_the_rule(rows, from_meta):
    """Two steps of 396 rows a task: below 800, the second step's weights come from the meta parameters; of 408: from the fp32 master, the
    same bits as with that asked for.  Against the oracle either way."""
    from paper_2401_04338_amd import GMeta
    from tests.helpers import small_cfg
    from tests.test_gpu_parity import TOL_BF16, _compare_step, _inputs
    cfg = small_cfg(n_tasks=4, n_support=rows, n_query=rows, n_fields=32, emb_dim=16, rows_per_field=300, bag_max=2, mlp_dtype=1,
                    layer_dims=(32 * 16 + 5, 1024, 256, 1))   # (millions of weights: some round the other way)
    sup, qry, params = _inputs(cfg)
    ctx = GMeta.from_config(cfg, workspace_bytes=1 << 30)
    out, _ = _compare_step(cfg, ctx, sup, qry, params, 2, 1, TOL_BF16, f"{rows} rows", operand="bf16")
    a = [x.clone() for x in out["dW"]]
    ctx.configure("theta_from_meta", 0)
    out, _ = _compare_step(cfg, ctx, sup, qry, params, 2, 1, TOL_BF16, f"{rows} rows, fp32 master", operand="bf16")
    ctx.close()
    assert all(torch.equal(x, y) for x, y in zip(a, out["dW"])) != from_meta
