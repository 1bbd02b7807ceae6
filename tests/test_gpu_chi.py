"""The chi kernel at the edges of its chunks and frequency blocks, with row
interchanges, extreme scales and singular chains, against LAPACK's pivoted
tridiagonal solve (the oracle).

Tolerance: both solvers are Gaussian elimination with partial pivoting, so
their results differ by at most 2 c u kappa(A) |n1| ||z|| ||x|| per frequency
(c = 8, u = 2^-53); A here is not normal, so kappa comes from its singular values.
"""
import numpy as np
import pytest

from oracle import chi as ochi

from gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    import torch
    import paper_2203_01120_amd as tm
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    tm.load()
    return tm


def coefficients(m, seed, pivots, scale=1.0):
    rng = np.random.default_rng(seed)
    a = 1e-3 if pivots else 1.0   # small diagonals force interchanges
    return dict(alpha=scale * a * (rng.standard_normal(m) + 0.1j * rng.standard_normal(m)),
                beta=scale * (0.5 + np.abs(rng.standard_normal(m))),
                gamma=scale * (rng.standard_normal(m) + 1j * rng.standard_normal(m)),
                z=rng.standard_normal((3, m)) + 1j * rng.standard_normal((3, m)),
                zn=rng.standard_normal(m) + 1j * rng.standard_normal(m), n1=1.7, steps_done=m)


def bound(co, m, omega, eta):
    T = ochi.tridiag(co, m)
    zn = np.linalg.norm(np.concatenate([co["zn"][None], co["z"]]), axis=1)
    out = np.zeros((4, len(omega)))
    for j, w in enumerate(omega):
        A = (w + 1j * eta) * np.eye(m) - T
        s = np.linalg.svd(A, compute_uv=False)
        x = np.linalg.solve(A, np.eye(m)[:, 0])
        out[:, j] = 16 * 2.0 ** -53 * s[0] / s[-1] * co["n1"] * zn * np.linalg.norm(x)
    return out


@pytest.mark.parametrize("scale", [1.0, 2.0 ** 450, 2.0 ** -450], ids=["1", "2^450", "2^-450"])
@pytest.mark.parametrize("pivots", [False, True], ids=["dominant", "interchanges"])
@pytest.mark.parametrize("m,nw", [(1, 1), (2, 15), (3, 16), (64, 17), (65, 63), (66, 5), (129, 64), (200, 33)])
def test_chi_against_lapack(lib, m, nw, pivots, scale):
    tm = lib
    say(f"chi m={m} nw={nw} pivots={pivots} scale={scale:.3g}")
    co = coefficients(m, 100 * m + nw, pivots, scale)
    omega, eta = scale * np.linspace(-1.5, 1.5, nw), scale * 0.05
    got = tm.tm_chi_tensor(co, m, omega, eta)
    unit = coefficients(m, 100 * m + nw, pivots)      # powers of two: the same numbers scaled exactly
    om1 = omega / scale
    ref = ochi.chi_lanczos(dict(unit, z=np.concatenate([unit["zn"][None], unit["z"]])), om1, 0.05, m)
    assert np.all(np.abs(got * scale - ref) <= bound(unit, m, om1, 0.05))
    assert np.array_equal(tm.tm_chi(co, m, omega, eta), got[1:])


def test_singular_chain_is_an_error(lib):
    tm = lib
    say("chi singular")
    m = 70
    co = coefficients(m, 1, False)
    co["alpha"][:], co["beta"][:], co["gamma"][:] = 0.5, 0.0, 0.0
    with pytest.raises(tm.TmError) as e:
        tm.tm_chi(co, m, np.array([0.25, 0.5]), 0.0)
    assert e.value.code == tm.TM_EINVAL
    assert np.isfinite(tm.tm_chi(co, m, np.array([0.25, 0.75]), 0.0)).all()
