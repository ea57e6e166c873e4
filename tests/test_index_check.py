"""The check of the indices (all that stands before the gathers) finds one bad index wherever it lies.  Tables of one size:
a workgroup's threads read eight indices a trip, `step` = 1024 x (workgroups of the (task, set)) apart, so the places are the ends of
some of the eight, of the trip after and of the list (and of trips of smaller workgroups).  Tables of different sizes: bag by bag.  gm_index_prep checks and does
not gather."""
from types import SimpleNamespace

import numpy as np
import pytest
import torch

from tests.test_gpu_parity import gm  # noqa: F401

pytestmark = pytest.mark.gpu
F, ROWS = 2, 50


def _set(samples, bag):
    n = samples * F
    return SimpleNamespace(n_samples=samples, task_offsets=np.array([0, samples], dtype=np.int64), labels=torch.zeros(samples, device="cuda:0"),
                           bag_offsets=torch.arange(0, (n + 1) * bag, bag, dtype=torch.int64, device="cuda:0"), nnz=n * bag,
                           indices=torch.arange(n * bag, dtype=torch.int32, device="cuda:0") % ROWS, dense=torch.zeros(samples, 1, device="cuda:0"))


@pytest.mark.parametrize("uneven", [0, 1])
@pytest.mark.parametrize("samples,bag,split", [(100, 6, 1), (300, 5, 2), (700, 9, 5)])   # (step = 256 x split: workgroups of 256 threads)
def test_one_bad_index(gm, samples, bag, split, uneven):  # noqa: F811
    from paper_2401_04338_amd import GMetaError
    step, n = 256 * split, samples * F * bag
    assert split == max(1, 2 * samples * F // 512) and n > 4 * step
    ctx = gm(F, [ROWS, ROWS + uneven], 4, 1, [F * 4 + 1, 8, 1], 0, workspace_bytes=1 << 26)
    sets = [_set(samples, bag), _set(samples, bag)]
    ctx.index_prep(*sets)
    for s in sets:
        for at in sorted({k * step + d for k in range(5) for d in (-1, 0, 1)} - {-1} | {n - 1}):
            if at >= n:
                continue
            good = int(s.indices[at])
            for bad in (-1, ROWS + uneven):
                s.indices[at] = bad
                with pytest.raises(GMetaError) as e:
                    ctx.index_prep(*sets)
                assert e.value.code == -2, (at, bad)
            s.indices[at] = good
    ctx.index_prep(*sets)
    ctx.close()


@pytest.mark.parametrize("uneven", [0, 1])
@pytest.mark.parametrize("small,large,bag", [(4, 4000, 3), (16, 1500, 9), (40, 16384, 1)])
def test_one_bad_index_beside_small_tasks(gm, small, large, bag, uneven):  # noqa: F811
    """The largest task decides how many workgroups every (task, set) gets: several here, of which the one-sample tasks fill one.  Their counts
    are cleared and added; a bad index is found at the ends of the large task's trips and in the tasks beside it."""
    from paper_2401_04338_amd import GMetaError
    sizes = [1] * (small // 2) + [large] + [1] * (small // 2)
    tasks, most = small + 1, 2 * large * F
    few, parts = min(most // 1024, 64 // tasks), min(most // 16384, 1024 // tasks)   # (the largest task is more than four times the average)
    split = max(few, parts)
    assert split > 1 and 4 * 2 * sum(sizes) * F < most * tasks
    ctx = gm(F, [ROWS, ROWS + uneven], 4, 1, [F * 4 + 1, 8, 1], 0, workspace_bytes=1 << 27)
    sets = [_set(sum(sizes), bag), _set(sum(sizes), bag)]
    for s in sets:
        s.task_offsets = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    clean = ctx.index_prep(*sets)
    per, step = F * bag, 1024 * split
    first, last = small // 2 * per, (small // 2 + large) * per   # the large task's lookups
    places = {0, first - 1, first, last - 1, last, sets[0].nnz - 1}
    places |= {first + k * step + d for k in (1, 7, 8, 9) for d in (-1, 0, 1) if k * step + d < last - first}
    for s in sets:
        for at in sorted(places):
            good = int(s.indices[at])
            s.indices[at] = -1
            with pytest.raises(GMetaError) as e:
                ctx.index_prep(*sets)
            assert e.value.code == -2, at
            s.indices[at] = good
    again = ctx.index_prep(*sets)
    assert all(torch.equal(clean[k], again[k]) for k in clean)
    ctx.close()


@pytest.mark.parametrize("uneven", [0, 1])
@pytest.mark.parametrize("samples,bag,split", [(400, 25, 1), (700, 14, 2), (1000, 16, 3)])
def test_one_bad_index_in_a_larger_task(gm, samples, bag, split, uneven):  # noqa: F811
    """1,024 threads, eight indices a trip (`step` apart), a workgroup a (task, set) or, from 2,048 bags of both sets on, several."""
    from paper_2401_04338_amd import GMetaError
    step, n = 1024 * split, samples * F * bag
    assert split == max(1, 2 * samples * F // 1024) and n > 8 * step
    ctx = gm(F, [ROWS, ROWS + uneven], 4, 1, [F * 4 + 1, 8, 1], 0, workspace_bytes=1 << 26)
    sets = [_set(samples, bag), _set(samples, bag)]
    ctx.index_prep(*sets)
    for s in sets:
        for at in sorted({k * step + d for k in (0, 1, 7, 8) for d in (-1, 0, 1)} - {-1} | {n - 1}):
            if at >= n:
                continue
            good = int(s.indices[at])
            s.indices[at] = ROWS + uneven
            with pytest.raises(GMetaError) as e:
                ctx.index_prep(*sets)
            assert e.value.code == -2, at
            s.indices[at] = good
    ctx.index_prep(*sets)
    ctx.close()
