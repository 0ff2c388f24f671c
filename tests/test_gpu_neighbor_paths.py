"""Branches of the list build that the other lists do not reach, bit for bit
against the brute-force oracle list: images outside the 32-bit sort keys
(atoms stored many cells away from home), rows sorted outside LDS (more than
512 neighbours), the multi-block scans, and a mostly empty box (coarse cells)."""
import numpy as np
import pytest

from oracle import brute_force_neighbors
from workloads import make_batch
from gpu_helpers import gpu, gpu_list_triples, need_gpu, oracle_triples

pytestmark = gpu


def _box(n, L, seed, spread=0):
    rng = np.random.default_rng(seed)
    pos = rng.uniform(0.0, L, (n, 3)) + L * rng.integers(-spread, spread + 1, (n, 3))
    return make_batch([(pos.astype(np.float32), rng.integers(0, 2, n).astype(np.int32), np.eye(3) * L, (1, 1, 1))])


@pytest.mark.parametrize("name,n,L,cutoff,spread", [
    ("far images", 300, 15.0, 5.0, 3),
    ("long rows", 700, 12.0, 7.0, 0),
    ("long rows, far images", 640, 12.0, 7.0, 4),
    ("sparse box", 60, 90.0, 5.0, 0),
])
def test_list_branches_bit_exact(name, n, L, cutoff, spread):
    g = need_gpu()
    batch = _box(n, L, 7, spread)
    print(f"neighbour list: {name} N={n} L={L} cutoff={cutoff}", flush=True)
    nl = g.build_neighbors(g.System.from_batch(batch, "cuda"), cutoff)
    ref = brute_force_neighbors(batch, cutoff)
    assert np.array_equal(gpu_list_triples(nl), oracle_triples(ref))
    rev = nl.rev[: nl.n_pairs].cpu().numpy()
    t = gpu_list_triples(nl)
    assert np.array_equal(t[rev, 0], t[:, 1]) and np.array_equal(t[rev, 1], t[:, 0])
    assert np.array_equal(t[rev, 2:], -t[:, 2:])


@pytest.mark.parametrize("n", [16384, 16385])
def test_scan_block_edge(n):
    """The last length one scan block walks over, and the first split one: row
    pointers are the running counts of a list whose rows are checked above."""
    g = need_gpu()
    L = (n / 0.05) ** (1.0 / 3.0)
    nl = g.build_neighbors(g.System.from_batch(_box(n, L, 3), "cuda"), 4.0)
    ptr = nl.row_ptr.cpu().numpy()
    assert ptr[0] == 0 and ptr[-1] == nl.n_pairs and np.all(np.diff(ptr) >= 0)
    t = gpu_list_triples(nl)
    rev = nl.rev[: nl.n_pairs].cpu().numpy()
    assert np.array_equal(t[rev, 0], t[:, 1]) and np.array_equal(t[rev, 1], t[:, 0])
