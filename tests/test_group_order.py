"""The order of grouped records over the spans of the numbers they are ordered by (none, one digit, several, more than 64 bits
together; either side of the line between comparing and counting digits), streams of zero and one record, and a workspace that
holds one of the two sets only."""
import numpy as np
import pytest
import torch

from oracle import maml_dlrm as O
from tests.helpers import small_cfg

pytestmark = pytest.mark.gpu
I64 = np.iinfo(np.int64)


@pytest.mark.parametrize("n,lo,hi,b_hi,share,ws", [
    (0, 0, 1, 1, (1, 2), 1 << 24), (1, 5, 6, 1, (1, 2), 1 << 24), (300, 7, 8, 1, (2, 3), 1 << 24), (999, -3, 8192, 2, (1, 2), 1 << 24),
    (1000, 0, 40, 9000, (0, 1), 1 << 24), (1000, I64.min, I64.max, 1, (1, 1), 1 << 24), (1000, I64.min, I64.max, 50, (1, 2), 1 << 24),
    (60000, 0, 300, 3, (1, 2), 1 << 20), (4000, I64.min, I64.max, 1, (1, 1), 1 << 24), (4000, I64.min, I64.max, 50, (1, 2), 1 << 24),
    (200, 0, 1 << 31, 1, (1, 2), 1 << 24), (600, 0, 1 << 31, 1, (1, 2), 1 << 24), (40, -5, 1 << 40, 3, (1, 2), 1 << 24)])
def test_orders(n, lo, hi, b_hi, share, ws):
    from paper_2401_04338_amd import GMeta
    F = 4
    cfg = small_cfg(n_fields=F)
    rng = np.random.default_rng(n + b_hi)
    ids = rng.integers(lo, hi, size=max(1, min(n // 3, 200)), dtype=np.int64)
    if hi == I64.max and n:
        ids[:2] = I64.min, I64.max
    task = rng.choice(ids, size=n) if n else np.zeros(0, np.int64)
    batch = rng.integers(0, b_hi, size=n).astype(np.int64)
    off = np.concatenate([[0], np.cumsum(rng.integers(0, 3, size=n * F))]).astype(np.int64)
    idx = rng.integers(0, 40, size=int(off[-1])).astype(np.int32)
    dense, labels = rng.standard_normal((n, cfg.n_dense)).astype(np.float32), rng.random(n).astype(np.float32)
    ref = O.group_batch(F, task, batch, off, idx, dense, labels, *share) if n else None
    ctx = GMeta.from_config(cfg, workspace_bytes=ws)
    dev = ctx.device
    got = ctx.group_batch(task, batch, *(torch.from_numpy(x).to(dev) for x in (off, idx, dense, labels)), *share)
    for g, s in zip(got, ref or (None, None)):
        if s is None:
            assert len(g.task_offsets) == 1 and len(g.labels) == 0
            continue
        d = g.numpy()
        for k in ("task_offsets", "bag_offsets", "indices", "dense", "labels"):
            assert np.array_equal(np.asarray(d[k]), np.asarray(s[k])), k
    ctx.close()
