"""fp32: the order in which the last layer's logits and the per-task column sums are added, bit for bit.  The adapted weights
follow from these sums, and a hidden unit near zero can fall on either side of it with their last bit."""
from types import SimpleNamespace

import numpy as np
import pytest
import torch

from tests.test_gpu_parity import gm  # noqa: F401

pytestmark = pytest.mark.gpu
D = 4   # one field of empty bags: its columns are zero


def _set(sizes, x, y):
    n = len(y)
    dev = "cuda:0"
    return SimpleNamespace(task_offsets=np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64), labels=torch.tensor(y, dtype=torch.float32, device=dev),
                           bag_offsets=torch.zeros(n + 1, dtype=torch.int64, device=dev), indices=torch.zeros(0, dtype=torch.int32, device=dev),
                           dense=torch.tensor(x, dtype=torch.float32, device=dev))


def _step(gm, sizes, x, y, w):  # noqa: F811
    n_dense = x.shape[1]
    ctx = gm(1, [3], D, n_dense, [D + n_dense, 1], 0, workspace_bytes=1 << 26)
    params = SimpleNamespace(emb=torch.zeros(3, D, device="cuda:0"), b=[torch.zeros(1, device="cuda:0")],
                             W=[torch.tensor(np.concatenate([np.zeros(D), w])[:, None], dtype=torch.float32, device="cuda:0")])
    qry = _set(sizes, x, y)
    out = ctx.meta_step(_set([1] * len(sizes), x[:len(sizes)], y[:len(sizes)]), qry, params, 0.1, 0, 1)
    got = {k: out[k].cpu().numpy() for k in ("task_loss",)} | {k: out[k][0].cpu().numpy() for k in ("dW", "db")}
    ctx.close()
    return got


@pytest.mark.parametrize("n_dense", [20, 75, 301])
def test_logits(gm, n_dense):  # noqa: F811
    """64 sums, one for every column modulo 64, in ascending columns; then halves are added.  2^24 + 1 is rounded to 2^24,
    so 2^24, 1 and -2^24 at three columns add up to 1 or to 0, as their order has it."""
    rng = np.random.default_rng(n_dense)
    T = 400
    x = np.zeros((T, n_dense), dtype=np.float32)
    for r in x:
        r[rng.choice(n_dense, 3, replace=False)] = [2.0 ** 24, 1.0, -2.0 ** 24]
    cols = np.zeros((T, (D + n_dense + 63) // 64 * 64), dtype=np.float32)
    cols[:, D:D + n_dense] = x
    part = np.zeros((T, 64), dtype=np.float32)
    for c in range(0, cols.shape[1], 64):
        part = part + cols[:, c:c + 64]
    while part.shape[1] > 1:
        h = part.shape[1] // 2
        part = part[:, :h] + part[:, h:]
    z = part[:, 0].astype(np.float64)
    assert set(z) == {0.0, 1.0}
    got = _step(gm, [1] * T, x, np.zeros(T), np.ones(n_dense))
    assert np.max(np.abs(got["task_loss"][:T] - np.log1p(np.exp(z)))) < 1e-5


@pytest.mark.parametrize("rows", [1, 8, 9, 16, 17, 31, 33, 129, 257, 1023, 1500])
def test_column_sums(gm, rows):  # noqa: F811
    """Four chains, rows 8 c .. 8 c + 7 of every 32 in chain c, every product rounded before it is added; then the chains in
    order.  With zero weights a row's delta is (1/2 - label) / rows."""
    rng = np.random.default_rng(rows)
    n_dense = 270
    x = rng.standard_normal((rows, n_dense)).astype(np.float32)
    y = (rng.random(rows) < 0.5).astype(np.float32)
    delta = (np.float32(0.5) - y) * (np.float32(1) / np.float32(rows))
    terms = np.concatenate([x * delta[:, None], delta[:, None]], axis=1)
    chains = np.zeros((4, n_dense + 1), dtype=np.float32)
    for s in range(rows):
        chains[s // 8 % 4] += terms[s]
    want = ((chains[0] + chains[1]) + chains[2]) + chains[3]
    got = _step(gm, [rows], x, y, np.zeros(n_dense))
    assert np.array_equal(got["dW"][D:, 0], want[:-1])
    assert np.array_equal(got["db"], want[-1:])


@pytest.mark.parametrize("bf", [0, 1])
@pytest.mark.parametrize("rows", [1, 4, 5, 8, 9, 16, 17, 33, 64, 65])
def test_a_large_task_beside(gm, bf, rows):  # noqa: F811
    """How many waves a launch of the sums has follows from the wave's largest task; what a small task gets from it does not."""
    rng = np.random.default_rng(rows)
    n_dense, big = 60, 200
    dims = [D + n_dense, 600, 40, 1]
    x, y = rng.standard_normal((rows + big, n_dense)).astype(np.float32), (rng.random(rows + big) < 0.5).astype(np.float32)
    params = SimpleNamespace(emb=torch.zeros(3, D, device="cuda:0"), b=[torch.tensor(rng.standard_normal(n), dtype=torch.float32, device="cuda:0") for n in dims[1:]],
                             W=[torch.tensor(rng.standard_normal((a, b)) / 4, dtype=torch.float32, device="cuda:0") for a, b in zip(dims[:-1], dims[1:])])
    ctx = gm(1, [3], D, n_dense, dims, bf, workspace_bytes=1 << 28)
    alone, beside = _set([rows], x[:rows], y[:rows]), _set([rows, big], x, y)
    a, b = (ctx.meta_step(s, s, params, 0.1, 2, 1) for s in (alone, beside))
    assert torch.equal(a["task_loss"][:1], b["task_loss"][:1])
    ctx.close()
