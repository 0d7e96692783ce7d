"""fp32 operands as three bf16 planes, modelled with numpy: what a product of two of them is off by, whole and with a piece missing.  The
limits that tests/test_gpu_fp32_planes.py sets for results lie between the two."""
import numpy as np
import pytest

SIX = [(2, 0), (0, 2), (1, 1), (1, 0), (0, 1), (0, 0)]   # planes of the first and of the second operand


def bf16(x):
    b = np.float32(x).view(np.uint32).astype(np.uint64)
    return ((b + 0x7fff + ((b >> 16) & 1)) & 0xffff0000).astype(np.uint32).view(np.float32)


def planes(x):
    p, rest = [], np.float32(x)
    for _ in range(3):
        p.append(bf16(rest).astype(np.float64))
        rest = np.float32(rest - bf16(rest))
    assert (rest == 0).all()
    return p


def product(x, y, products=SIX, keep=(3, 3)):
    a, b = planes(x), planes(y)
    return sum(a[i] * b[j] for i, j in products if i < keep[0] and j < keep[1])


def error(got, want):
    return np.linalg.norm(got - want) / np.linalg.norm(want)


def operands(seed):
    rng = np.random.default_rng(seed)
    return [np.float32(rng.standard_normal(20000)) for _ in range(2)]


def test_planes_hold_every_bit():
    x, y = operands(1)
    for v in (x, y * np.float32(2.0 ** -125), np.float32([2.0 ** -149, -(2.0 ** 111), 1 + 2.0 ** -23, 1 + 2.0 ** -8 - 2.0 ** -23])):
        up = v * np.float32(2.0 ** 16)   # as the kernels split it
        assert (sum(planes(up)) == v.astype(np.float64) * 2.0 ** 16).all()


def test_products_left_out():
    x, y = operands(2)
    worst = np.float32(1 + 2.0 ** -8 - 2.0 ** -17 + np.arange(-64, 64) * 2.0 ** -23)
    for a, b in ((x, y), (worst.repeat(128), np.tile(worst, 128))):
        want = a.astype(np.float64) * b
        assert np.abs(product(a, b) / want - 1).max() <= 2.0 ** -24 * (1 + 2.0 ** -9)
    assert error(product(x, y), x.astype(np.float64) * y) <= 4e-8


@pytest.mark.parametrize("missing", SIX)
def test_a_missing_product_shows(missing):
    x, y = operands(3)
    assert error(product(x, y, [p for p in SIX if p != missing]), x.astype(np.float64) * y) >= 2e-6


@pytest.mark.parametrize("keep", [(2, 3), (3, 2)])
def test_a_missing_last_plane_shows(keep):
    x, y = operands(4)
    assert error(product(x, y, keep=keep), x.astype(np.float64) * y) >= 2e-6
