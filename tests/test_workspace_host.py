"""Workspace sizes (host-only C code): the double backward keeps partial products
for the row chunks it uses and the invariants' adjoints in their place, and
force variance takes nothing besides the per-head arrays."""
import ctypes as C

import pytest

from paper_2505_22168_amd import _capi as A
from test_plan_host import _Sys, _model

F, FP = 360, 384


def _bytes(op, hidden, n, heads=1, flags=0, pairs_per_atom=60):
    nl = A.gmnn_neighbors()
    nl.capacity, nl.cutoff = pairs_per_atom * n, 5.0
    return A.load().gmnn_workspace_bytes(op, C.byref(_model(hidden=hidden, heads=heads)), C.byref(_Sys([n]).c), C.byref(nl),
                                         flags)


@pytest.mark.parametrize("hidden", [256, 512])
@pytest.mark.parametrize("flags", [0, A.GMNN_PREC_BF16])
@pytest.mark.parametrize("n", [11200, 100000])
def test_backward_workspace(hidden, flags, n):
    # per atom, in words: four moment arrays, X1 and three hidden arrays of two rows, W3's rows, and
    # the larger of the adjoints of the invariants and the partials of chunks of 512 rows; the
    # per-pair position gradients; 2% and 8 MB for the sums over atoms
    rows = 400 + 2 * FP + 6 * hidden + hidden + 1
    shared = max(2 * FP, (FP + hidden) * hidden / 256)
    assert _bytes(A.GMNN_OP_BACKWARD, hidden, n, flags=flags) < 1.02 * (4 * n * (rows + shared) + 720 * n) + (8 << 20)


@pytest.mark.parametrize("heads", [6, 16])
def test_force_variance_workspace(heads):
    # per-pair gradients and moment gradients of every head, and what one head needs
    n = 11200
    one, many = (_bytes(A.GMNN_OP_ENERGY_FORCES, 256, n, heads=heads, flags=f) for f in (0, A.GMNN_WANT_FORCE_VAR))
    assert many - one <= (heads - 1) * (400 * n + 720 * n + 512)


def test_noalloc_limit_with_force_variance():
    """3270 atoms with 60 neighbours and 15 heads fit the fixed scratch array."""
    assert _bytes(A.GMNN_OP_ENERGY_FORCES, 256, 3270, heads=15, flags=A.GMNN_WANT_FORCE_VAR) <= 64 << 20
