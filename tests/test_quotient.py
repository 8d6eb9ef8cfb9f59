"""The quotient of two binary32 numbers from a product in binary64 with the
divisor's reciprocal, as the kernels that index voxels and place free samples
take it, against the division rounded once: equal wherever the product is at
least 2^-120 in magnitude (below that the kernels divide)."""
import numpy as np
import pytest


def product(a, b):
    return a.astype(np.float64) * (1.0 / b.astype(np.float64))


def check(a, b):
    q = product(a, b)
    big = np.abs(q) >= 2.0 ** -120
    with np.errstate(over="ignore"):
        got, want = q.astype(np.float32)[big], (a / b)[big]
    assert np.array_equal(got.view(np.uint32), want.view(np.uint32))
    return int(big.sum())


@pytest.mark.parametrize("seed", range(4))
def test_random_quotients(seed):
    rng = np.random.default_rng(seed)
    bits = rng.integers(0, 0x7F800000, size=(2, 400_000), dtype=np.uint32)
    a, b = bits.view(np.float32)
    b = np.maximum(b, np.float32(1e-30))
    a *= rng.choice(np.array([-1, 1], np.float32), a.shape)
    assert check(a, b) > 100_000


@pytest.mark.parametrize("res", [0.05, 0.1, 0.2, 0.25, 0.3, 1.0 / 3.0, 0.3002929985523224, 7.0])
def test_quotients_next_to_midpoints(res):
    # numerators nearest to (a midpoint of binary32) x (the divisor), and their
    # neighbours: the quotients closest to where the rounding turns
    b = np.float32(res)
    rng = np.random.default_rng(int(1000 * res))
    m = (rng.integers(1 << 24, 1 << 25, 200_000) | 1).astype(np.float64)
    m *= 2.0 ** rng.integers(-40, 0, m.shape)
    a = (m * float(b)).astype(np.float32)
    a = np.concatenate([a, np.nextafter(a, np.float32(0)), np.nextafter(a, np.float32(np.inf)), -a])
    assert check(a, np.full_like(a, b)) > 500_000
