"""Parts of a four-step pass (CPU model of the tile kernel's rules): in a tile
below its mirror, which of a thread's 16 entries are read or stored at their
mirror follows from the points of the group's earlier stages alone."""
import itertools

import pytest


def _mirror(x):
    m = 0x5555555555555555
    return ((x & m) << 1) | ((x >> 1) & m)


def _md(d):
    return (0, 2, 1, 3)[d]


def _strides(j, k):
    """Strides of the digits d0 .. d3 and m after j stages, L = k + 6."""
    L = k + 6
    return [4 ** (L - j + p) if p < j else 4 ** (p - j) for p in range(4)], 4 ** (4 - j)


K = 2
TILES = [h for h in range(4 ** K) if h < _mirror(h)]


@pytest.mark.parametrize("s0", [1, 2, 3])
def test_read_rule(s0):
    sd, sm = _strides(s0, K)
    for hi, w, a, b, r in itertools.product(TILES, range(16), range(4), range(4), range(16)):
        q, p = r % 4, r // 4
        rm = _md(q) + 4 * _md(p)
        if s0 == 3:      # lane (w0, w1, o0), wave o1, registers (o2, d3)
            i = (16 * hi + w) * sm + a * sd[0] + b * sd[1] + q * sd[2] + p * sd[3]
            direct = q == 1 or (q != 2 and a + 4 * b <= _md(a) + 4 * _md(b))
        else:            # lane (d2, d3, w0), wave w1, registers (o0, d1) or (o0, o1)
            i = (16 * hi + w) * sm + a * sd[2] + b * sd[3] + q * sd[0] + p * sd[1]
            direct = q != 2 if s0 == 1 else r <= rm
        assert direct == (i < _mirror(i))


@pytest.mark.parametrize("s1", [1, 2, 3, 4])
def test_store_rule(s1):
    sd, sm = _strides(s1, K)
    for hi, a, b, c, r in itertools.product(TILES, range(4), range(4), range(16), range(16)):
        q, p = r % 4, r // 4
        rm = _md(q) + 4 * _md(p)
        if s1 == 1:      # lane (d1, d2, w0), wave w1, registers (o0, d3)
            y = (16 * hi + c) * sm + a * sd[1] + b * sd[2] + q * sd[0] + p * sd[3]
            direct = q != 2
        elif s1 == 2:    # lane (d2, d3, w0), wave w1, registers (o0, o1)
            y = (16 * hi + c) * sm + a * sd[2] + b * sd[3] + q * sd[0] + p * sd[1]
            direct = r <= rm
        else:
            o01 = a + 4 * b
            ok = o01 <= _md(a) + 4 * _md(b)
            if s1 == 3:  # lane (d3, w0, o0), wave o1, registers (o2, w1)
                y = (16 * hi + c // 4 + 4 * p) * sm + c % 4 * sd[3] + a * sd[0] + b * sd[1] + q * sd[2]
                direct = q == 1 or (q != 2 and ok)
            else:        # lane (w0, w1, o0), wave o1, registers (o2, o3)
                y = (16 * hi + c) * sm + a * sd[0] + b * sd[1] + q * sd[2] + p * sd[3]
                direct = r < rm or (r == rm and ok)
        assert direct == (y < _mirror(y))


def test_rows_of_four_real_coefficients():
    # the oldest point's row of the off-diagonal points: the phase e^{-i phi} in
    # the thread's factor, the rest on sums and differences of the four entries
    import numpy as np
    rng = np.random.default_rng(8)
    for _ in range(50):
        s, eta, x = rng.normal(size=2), complex(*rng.normal(size=2)), rng.normal(size=4) + 1j * rng.normal(size=4)
        D = s[0] - s[1]
        phi, th, g = D * eta.imag * (s[0] + s[1]), D * D * eta.imag, D * D * eta.real
        p, q = x[0] + x[3], x[0] - x[3]
        row1 = np.cos(th) * p - 1j * np.sin(th) * q + np.exp(-g) * x[1] + np.exp(g) * x[2]
        row2 = np.cos(th) * p + 1j * np.sin(th) * q + np.exp(-g) * x[2] + np.exp(g) * x[1]
        for (a, b), got in (((0, 1), np.exp(-1j * phi) * row1), ((1, 0), np.exp(1j * phi) * row2)):
            F = [np.exp(-(s[a] - s[b]) * (eta * s[c] - np.conj(eta) * s[d])) for c in (0, 1) for d in (0, 1)]
            assert abs(got - np.dot(F, x)) <= 1e-13 * np.abs(F).max() * np.abs(x).sum()
