"""Selection launches at their edges, bit for bit against the oracle: several
feature chunks, more rows than the blocks take at once, more training rows
than a block stages, exact ties."""
import numpy as np
import pytest
import torch

from oracle.bal import max_distance_selection
from gpu_helpers import gpu, need_gpu

pytestmark = gpu


@pytest.mark.parametrize("n,d,t,b", [(16, 288, 0, 5), (17, 289, 0, 5), (40, 600, 17, 6), (33, 5, 40, 8),
                                     (8193, 3, 0, 3), (8209, 2, 18, 3)])
def test_selection_paths(n, d, t, b):
    g = need_gpu()
    rng = np.random.default_rng(n + d)
    pool = rng.normal(size=(n, d))
    pool[n // 2] = pool[1]   # an exact tie: the smaller index first
    train = rng.normal(size=(t, d)) if t else None
    print(f"selection n={n} d={d} t={t}", flush=True)
    got = g.select_max_distance(torch.as_tensor(pool, device="cuda"), b,
                                None if train is None else torch.as_tensor(train, device="cuda")).cpu().numpy()
    assert np.array_equal(got, max_distance_selection(pool, b, train))
