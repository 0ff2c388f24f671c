"""A cell far from reduced: two atoms of a cubic lattice (4.6 A) described by
lattice vectors that are long integer combinations of its own, so that the
stencil has 6.3 million runs of cells (above 2^22 their quotients by FP32
reciprocals are no longer exact).  The list is the reduced lattice's with the
images transformed, each pair under the inclusion test of the definition."""
import numpy as np

from workloads import make_batch
from gpu_helpers import gpu, gpu_list_triples, need_gpu

pytestmark = gpu

A, CUTOFF = 4.6, 5.0
V = np.array([[-44, 67, -92], [35, -60, 71], [5, -9, 10]])  # reduced image n = image n V of the long cell
POS = np.array([[0.0, 0.0, 0.0], [3.79307720, 1.41937617, 3.93932207]], np.float32)


def _expected(cell):
    n = np.array(list(np.ndindex(7, 7, 7))) - 3
    S, x, rows = n @ V, POS.astype(np.float64), []
    for i in range(2):
        for j in range(2):
            d = (x[j] - x[i]) + ((S[:, :1] * cell[0] + S[:, 1:2] * cell[1]) + S[:, 2:] * cell[2])
            d2 = (d[:, 0] * d[:, 0] + d[:, 1] * d[:, 1]) + d[:, 2] * d[:, 2]
            rows += [(i, j, *s) for s, r in zip(S, d2) if 0.0 < r < CUTOFF * CUTOFF]
    return np.array(sorted(rows))


def test_skewed_cell_list():
    g = need_gpu()
    U = np.rint(np.linalg.inv(V)).astype(np.int64)
    assert np.array_equal(U @ V, np.eye(3, dtype=np.int64))
    cell = U * A
    print("neighbour list of a cell far from reduced", flush=True)
    nl = g.build_neighbors(g.System.from_batch(make_batch([(POS, np.array([0, 1], np.int32), cell, (1, 1, 1))]), "cuda"),
                           CUTOFF)
    t = gpu_list_triples(nl)
    assert np.array_equal(t, _expected(cell))
    rev = nl.rev[: nl.n_pairs].cpu().numpy()
    assert np.array_equal(t[rev, 0], t[:, 1]) and np.array_equal(t[rev, 2:], -t[:, 2:])
