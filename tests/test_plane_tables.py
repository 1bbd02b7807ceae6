"""The tables and row orders of the matrix-core plane kernels as the library
builds them (mx_constants, mx_twists and the row functions of plane.h, read by a
small host program linked with libtm.so) against the plain DFT.

Tolerance: sums of at most 47 terms of modulus one, 1e-13 of the inputs' sum.
"""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2203_01120_amd")

PROGRAM = r"""
#include <cstdio>
#include "plane.h"
using namespace tml;
int main() {
    auto row = [](const char* name, int n, auto count, auto value) {
        std::printf("%s %d", name, n);
        for (int i = 0; i < (int)count; ++i) std::printf(" %.17g", (double)value(i));
        std::printf("\n");
    };
    for (int n = 4; n <= kMxSide; ++n) {
        const std::vector<double2> c = mx_constants(n), t = mx_twists(n);
        row("stride", n, 1, [&](int) { return mx_stride(n); });
        row("cos", n, c.size(), [&](int i) { return c[i].x; });
        row("sin", n, c.size(), [&](int i) { return c[i].y; });
        row("twist_re", n, t.size(), [&](int i) { return t[i].x; });
        row("twist_im", n, t.size(), [&](int i) { return t[i].y; });
        row("partner", n, mx_pairs(n), [&](int j) { return mx_partner(n, j); });
        row("base", n, mx_steps(n), [&](int s) { return mx_partner_base(n, 4 * s); });
    }
    for (int n : {8, 20, 24, 32, 48}) {
        row("resident", n, n / 4, [&](int s) { return mx_resident_row(n, 4 * s); });
        const CPlan p = cplan(n);
        row("radices", n, p.nrad, [&](int s) { return p.rad[s]; });
    }
}
"""


@pytest.fixture(scope="module")
def tables(tmp_path_factory):
    from paper_2203_01120_amd import build_lib
    if not os.path.exists(build_lib.OUT):
        build_lib.build()
    d = tmp_path_factory.mktemp("plane_tables")
    src, exe = d / "tables.hip", d / "tables"
    src.write_text(PROGRAM)
    cmd = [build_lib._hipcc(), "--offload-host-only", "-O1", "-std=c++17", "-I", build_lib.CSRC, str(src), "-o", str(exe),
           "-L", PKG, "-l:libtm.so", f"-Wl,-rpath,{PKG}"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    out = {}
    for line in subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout.splitlines():
        name, n, *v = line.split()
        out[name, int(n)] = np.array([float(x) for x in v])
    return out


@pytest.mark.parametrize("n", range(4, 65))
def test_pairs_equal_the_dft(tables, n):
    stride = int(tables["stride", n][0])
    c, s = (tables[name, n].reshape(24, stride) for name in ("cos", "sin"))
    twist = tables["twist_re", n] + 1j * tables["twist_im", n]
    partner = tables["partner", n].astype(int)
    h = len(partner)
    assert h == (n + 1) // 2 and stride % 2 == 1 and stride >= h
    assert np.all(c[:, h:] == 0) and np.all(s[:, h:] == 0)     # K steps past the last pair add nothing
    both = np.concatenate([np.arange(h), partner[1:] if n % 2 else partner])
    assert sorted(both) == list(range(n))                       # every row once
    rng = np.random.default_rng(n)
    for reach in range(0, min(23, (n - 1) // 2) + 1):
        cm, sm, tw = c[:reach + 1, :h], s[:reach + 1, :h], twist[:reach + 1]
        m = np.arange(-reach, reach + 1)
        x = rng.standard_normal(2 * reach + 1) + 1j * rng.standard_normal(2 * reach + 1)
        p, q = x[reach:] * tw, x[reach::-1] * tw.conj()
        q[0] = 0
        C, S = (p + q) @ cm, (p - q) @ sm
        got = np.empty(n, complex)
        got[partner] = C - 1j * S
        got[:h] = C + 1j * S
        ref = np.exp(2j * np.pi * np.outer(np.arange(n), m) / n) @ x
        assert np.abs(got - ref).max() <= 1e-13 * (1 + np.abs(x).sum())
        f = rng.standard_normal(n) + 1j * rng.standard_normal(n)
        a, b = f[:h].copy(), f[partner].copy()
        if n % 2 == 1:
            b[0] = 0
        C, S = cm @ (a + b), sm @ (a - b)
        ref = np.exp(-2j * np.pi * np.outer(m, np.arange(n)) / n) @ f
        assert np.abs((C - 1j * S) * tw.conj() - ref[reach:]).max() <= 1e-13 * np.abs(f).sum()
        assert np.abs(((C + 1j * S) * tw)[1:] - ref[:reach][::-1]).max(initial=0.0) <= 1e-13 * np.abs(f).sum()


@pytest.mark.parametrize("n", range(4, 65))
def test_partners_of_a_step(tables, n):
    """The lanes of a K step find their partners at fixed distances from one row."""
    partner = tables["partner", n].astype(int)
    for step, base in enumerate(tables["base", n].astype(int)):
        for k in range(4):
            j = 4 * step + k
            if j >= len(partner):
                continue
            if n % 2 == 1 and step == 0:
                assert partner[j] == base + (0 if k == 0 else n - k)
            else:
                assert partner[j] == base + 3 - k
        assert 0 <= base < n


@pytest.mark.parametrize("n", [8, 20, 24, 32, 48])
def test_resident_rows_are_the_digit_reversed_positions(tables, n):
    """The rows that the kernels read against the positions of an in-place
    transform with the library's radices."""
    radices = tables["radices", n].astype(int)
    assert radices[0] == 4 and np.prod(radices) == n

    def position(i):   # of element i in a digit-reversed line
        pos, place = 0, n
        for r in radices:
            place //= r
            pos += i % r * place
            i //= r
        return pos

    rows = tables["resident", n].astype(int)
    for step, row in enumerate(rows):
        assert [position(4 * step + k) for k in range(4)] == [row + k * (n // 4) for k in range(4)]
    for base in tables["base", n].astype(int):   # partners are read from whole steps too
        assert base % 4 == 0 and base // 4 < len(rows)
