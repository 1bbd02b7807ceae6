"""The pruned transforms of the matrix-core plane kernels, restated in numpy and
compared with the plain DFT for every plane side and every reach that the
kernels take; and the rows of the resident ground state they read.

Tolerance: sums of at most 47 terms of modulus one, 1e-13 absolute.
"""
import numpy as np
import pytest


def _tables(n, reach):
    h, m = (n + 1) // 2, np.arange(reach + 1)
    j = np.arange(h)[:, None]
    ang = 2 * np.pi * ((j + 0.5) if n % 2 == 0 else j) * m / n
    twist = np.exp(-1j * np.pi * m / n) if n % 2 == 0 else np.ones(reach + 1)
    partner = (n - 1 - np.arange(h)) if n % 2 == 0 else np.where(np.arange(h) == 0, 0, n - np.arange(h))
    return np.cos(ang), np.sin(ang), twist, partner


@pytest.mark.parametrize("n", range(4, 65))
def test_pruned_pairs_equal_the_dft(n):
    rng = np.random.default_rng(n)
    for reach in range(0, min(23, (n - 1) // 2) + 1):
        c, s, tw, partner = _tables(n, reach)
        h = len(partner)
        m = np.arange(-reach, reach + 1)
        x = rng.standard_normal(2 * reach + 1) + 1j * rng.standard_normal(2 * reach + 1)
        # inverse: sums and differences of +m and -m, twisted
        p = x[reach:] * tw
        q = x[reach::-1] * tw.conj()
        q[0] = 0
        C, S = c @ (p + q), s @ (p - q)
        got = np.zeros(n, complex)
        got[partner] = C - 1j * S
        got[np.arange(h)] = C + 1j * S
        ref = np.exp(2j * np.pi * np.outer(np.arange(n), m) / n) @ x
        assert np.abs(got - ref).max() <= 1e-13 * (1 + np.abs(x).sum())
        # forward, of any real-space values
        f = rng.standard_normal(n) + 1j * rng.standard_normal(n)
        a, b = f[:h].copy(), f[partner].copy()
        if n % 2 == 1:
            b[0] = 0
        C, S = c.T @ (a + b), s.T @ (a - b)
        plus, minus = (C - 1j * S) * tw.conj(), (C + 1j * S) * tw
        ref = np.exp(-2j * np.pi * np.outer(m, np.arange(n)) / n) @ f
        assert np.abs(plus - ref[reach:]).max() <= 1e-13 * np.abs(f).sum()
        assert np.abs(minus[1:] - ref[:reach][::-1]).max(initial=0.0) <= 1e-13 * np.abs(f).sum()


@pytest.mark.parametrize("n", [8, 20, 24, 32, 48])
def test_resident_rows_are_the_digit_reversed_positions(n):
    radices, rest = [], n
    for r in (4, 5, 3, 2):
        while rest % r == 0:
            radices.append(r)
            rest //= r

    def position(i):   # of element i in a digit-reversed line
        pos, place = 0, n
        for r in radices:
            place //= r
            pos += i % r * place
            i //= r
        return pos

    def row(j0):       # of j0, a multiple of 4: the digits of j0 / 4 reversed
        d, w, pos = j0 // 4, n // 4, 0
        for r in radices[1:]:
            w //= r
            pos += d % r * w
            d //= r
        return pos

    for j0 in range(0, n, 4):
        assert [position(j0 + k) for k in range(4)] == [row(j0) + k * (n // 4) for k in range(4)]
