"""The three-operation division of the learned drift's inputs (quality_points in
graph_kernels.hip: q0 = a r with r = 1 / b rounded, e = a - q0 b and q0 + e r
fused) against the correctly rounded quotient, in float32 arithmetic made from
float64 that loses nothing: random significands, and quotients as near the
middle between two floats as two significands allow, where a rounding of the
correction itself would show."""
import numpy as np

F = np.float32


def fma32(x, y, z):
    """x y + z rounded once to float32 (normal range): x y is exact in float64,
    the sum's rounding error is kept (two-sum) and decides float32 ties."""
    p, z = x.astype(np.float64) * y.astype(np.float64), z.astype(np.float64)
    s = p + z
    t = s - p
    err = (p - (s - t)) + (z - t)
    f = s.astype(F)
    off = s - f.astype(np.float64)
    other = np.nextafter(f, np.where(off > 0, F(np.inf), F(-np.inf)))
    tie = (off != 0) & (np.abs(off) * 2 == np.abs(other.astype(np.float64) - f))
    return np.where(tie & (np.sign(err) == np.sign(off)) & (err != 0), other, f)


def three_operations(a, b):
    r = F(1) / b
    q0 = a * r
    return fma32(fma32(-q0, b, a), r, q0)


def test_random_significands():
    rng = np.random.default_rng(1)
    a = rng.integers(1 << 23, 1 << 24, 2_000_000).astype(F)
    b = rng.integers(1 << 23, 1 << 24, a.size).astype(F)
    b[:4096] = F((1 << 24) - 1) - np.arange(4096, dtype=F)  # where r a is furthest off
    a[:64] = F((1 << 24) - 1) - np.arange(64, dtype=F)
    assert np.array_equal(three_operations(a, b), a / b)


def test_quotients_next_to_the_middle_of_two_floats():
    """a 2^k = b M + d for odd M of 25 bits (the middle between two floats of
    the quotient) and small odd d, solved for a: M = -d / b modulo 2^k."""
    rng = np.random.default_rng(2)
    seen = 0
    for k in (24, 25):
        for d in (-7, -5, -3, -1, 1, 3, 5, 7):
            b = rng.integers(1 << 22, 1 << 23, 200_000, dtype=np.uint64) * 2 + 1
            b[:2048] = (1 << 24) - 1 - 2 * np.arange(2048, dtype=np.uint64)
            mod = np.uint64((1 << k) - 1)
            inv = b.copy()
            for _ in range(5):  # Newton: the inverse of b modulo 2^64
                inv *= np.uint64(2) - b * inv
            m = (np.uint64((-d) % (1 << 64)) * inv) & mod
            if k == 24:
                m |= np.uint64(1 << 24)
            prod = (b * m).astype(np.int64) + d
            a = prod >> k
            ok = (m >> np.uint64(24) == 1) & (a >= 1 << 23) & (a < 1 << 24)
            assert np.all(a << k == prod)
            a, b = a[ok].astype(F), b[ok].astype(F)
            assert np.array_equal(three_operations(a, b), a / b), (k, d)
            seen += a.size
    assert seen > 500_000
