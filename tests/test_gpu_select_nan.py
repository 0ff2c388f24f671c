"""Selection from pools and training sets with NaN features (a diverged model):
every pick is a row of the pool, picks are distinct, rows with a distance come
first and in the order they have without the others."""
import numpy as np
import pytest
import torch

from oracle.bal import max_distance_selection
from gpu_helpers import gpu, need_gpu

pytestmark = gpu

N, D = 37, 5


def _pick(g, pool, b, train=None):
    t = None if train is None else torch.as_tensor(train, device="cuda")
    return g.select_max_distance(torch.as_tensor(pool, device="cuda"), b, t).cpu().numpy().tolist()


@pytest.mark.parametrize("t", [0, 3, 20])
def test_pool_of_nan(t):
    g = need_gpu()
    print(f"selection from a pool of NaN, t={t}", flush=True)
    train = np.random.default_rng(t).normal(size=(t, D)) if t else None
    assert _pick(g, np.full((N, D), np.nan), 6, train) == list(range(6))


@pytest.mark.parametrize("bad", [[0], [36], [3, 17, 18]])
def test_some_nan_rows_come_last(bad):
    g = need_gpu()
    print(f"selection with NaN rows {bad}", flush=True)
    rng = np.random.default_rng(len(bad))
    pool = rng.normal(size=(N, D))
    pool[bad, 2] = np.nan
    good = np.setdiff1d(np.arange(N), bad)
    got = _pick(g, pool, N)
    assert got[: len(good)] == good[max_distance_selection(pool[good], len(good))].tolist()
    assert got[len(good):] == bad


def test_training_set_of_nan():
    """No entry has a distance at first (the smallest index is taken); from the first pick on all have."""
    g = need_gpu()
    print("selection against a training set of NaN", flush=True)
    pool = np.random.default_rng(1).normal(size=(N, D))
    got = _pick(g, pool, 8, np.full((4, D), np.nan))
    assert got == [0] + [int(k) + 1 for k in max_distance_selection(pool[1:], 7, pool[:1])]
    assert _pick(g, pool, 8, np.concatenate([np.full((1, D), np.nan), pool[:1]])) == max_distance_selection(
        pool, 8, pool[:1]).tolist()
