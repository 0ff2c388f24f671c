"""The three-part BF16 form of FP32 products (parts and bound as stated beside
the kernels), restated on the CPU: the parts add up to the value over the stated
range, and the three part products left out are at most 2^-24 of a term, with
operands that reach half of that and more."""
import numpy as np
import pytest
import torch


def _bf16(x):
    return torch.as_tensor(x, dtype=torch.float32).to(torch.bfloat16).to(torch.float32).numpy()


def _parts(v):
    v = np.asarray(v, np.float32)
    h = _bf16(v)
    m = _bf16(v - h)
    return h, m, _bf16(v - h - m)


def _mantissas():
    """Values in [1, 2): random, around every rounding edge of the first part, and the worst known."""
    rng = np.random.default_rng(1)
    edges = (1 + np.arange(128)[:, None] / 128 + 2.0 ** -8 + np.array([-1, 0, 1])[None] * 2.0 ** -17
             * np.array([1, 1, 1])).ravel()
    x = np.concatenate([rng.uniform(1, 2, 20000), edges, [1 + 2.0 ** -8 - 2.0 ** -17, 2 - 2.0 ** -23, 1 + 2.0 ** -23]])
    return x.astype(np.float32)


@pytest.mark.parametrize("exponent", [-103, -60, 0, 60, 126])
def test_parts_add_up(exponent):
    v = np.ldexp(_mantissas(), exponent)
    for s in (1, -1):
        h, m, l = _parts(s * v)
        assert np.array_equal(h.astype(np.float64) + m + l, s * v.astype(np.float64))


def test_largest_exact_value_and_beyond():
    edge = np.float32(3.396e38)  # below the midpoint of the largest bf16 value and infinity
    h, m, l = _parts([edge])
    assert h[0].astype(np.float64) + m[0] + l[0] == np.float64(edge)
    with np.errstate(all="ignore"):
        for v in (np.float32(3.4e38), np.float32(np.inf)):
            assert not np.isfinite(sum(p.astype(np.float64) for p in _parts([v])))[0]


def test_dropped_products():
    v = _mantissas()
    rng = np.random.default_rng(2)
    x = np.concatenate([v, v, v[-3:], v[-3:]])
    y = np.concatenate([rng.permutation(v), v, v[-3:], v[[-1, -3, -2]]])
    (_, mx, lx), (_, my, ly) = ([p.astype(np.float64) for p in _parts(a)] for a in (x, y))
    dropped = np.abs(mx * ly + lx * my + lx * ly) / (x.astype(np.float64) * y)
    assert dropped.max() <= 2.0 ** -24
    assert dropped.max() > 0.9 * 2.0 ** -24  # half an ulp is reached
