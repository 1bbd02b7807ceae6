"""chi for inputs that the one-sweep kernel does not answer for: infinite and far
frequencies, coefficients many orders apart, and poles of an undamped chain.
None of them may change what the other frequencies of the call get.

Tolerances: far from the spectrum chi = n1 z_1 / omega up to terms 1e-150 times
smaller, four roundings; an element of 1e160 on the diagonal cuts the chain off
there, so the result is the shorter chain's within the forward-error bound of
two eliminations; everything else is bit for bit.
"""
import numpy as np
import pytest

from gpu_util import say
from test_gpu_chi import bound, coefficients

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    import torch
    import paper_2203_01120_amd as tm
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    tm.load()
    return tm


@pytest.mark.parametrize("m", [1, 2, 65, 130])
def test_far_and_infinite_frequencies(lib, m):
    tm = lib
    say(f"chi far frequencies m={m}")
    co = coefficients(m, 7, False)
    near = np.linspace(-1.0, 1.0, 19)
    far = np.array([1e170, -1e200, 1e300, np.inf, -np.inf])
    alone = tm.tm_chi_tensor(co, m, near, 0.05)
    assert np.isfinite(alone).all()
    got = tm.tm_chi_tensor(co, m, np.concatenate([near[:10], far, near[10:], [np.nan]]), 0.05)
    assert np.array_equal(got[:, np.r_[0:10, 15:24]], alone)
    z1 = np.concatenate([co["zn"][None], co["z"]])[:, :1]
    ref = co["n1"] * z1 / far[:3]
    assert np.all(np.abs(got[:, 10:13] - ref) <= 2.0 ** -51 * np.abs(ref))
    assert np.all(got[:, 13:15] == 0)
    assert np.isnan(got[:, -1]).all()


def test_residual_coupling_is_not_used(lib):
    """The last beta and gamma couple to the step after the chain's end."""
    tm = lib
    say("chi last beta and gamma")
    m = 70
    co = coefficients(m, 8, False)
    omega = np.linspace(-1.0, 1.0, 5)
    ref = tm.tm_chi_tensor(co, m, omega, 0.05)
    for big in (1e200, np.inf, np.nan):
        other = dict(co, beta=co["beta"].copy(), gamma=co["gamma"].copy())
        other["beta"][-1] = big
        other["gamma"][-1] = big
        assert np.array_equal(tm.tm_chi_tensor(other, m, omega, 0.05), ref), big


@pytest.mark.parametrize("m,cut", [(2, 1), (90, 40), (90, 66)])
def test_chain_cut_by_a_large_element(lib, m, cut):
    tm = lib
    say(f"chi chain cut m={m} at {cut}")
    co = coefficients(m, 9, False)
    omega = np.linspace(-1.0, 1.0, 18)
    ref = tm.tm_chi_tensor(co, cut, omega, 0.05)
    tol = bound({k: (v[..., :cut] if np.ndim(v) else v) for k, v in co.items()}, cut, omega, 0.05)
    co["alpha"][cut] = 1e160
    got = tm.tm_chi_tensor(co, m, omega, 0.05)
    assert np.all(np.abs(got - ref) <= tol)


@pytest.mark.parametrize("alpha,beta,gamma", [
    ([-3.0, 2.0], [3.0], [-2.0]),
    ([0.0, 0.0, 0.0], [1.0, 1.0], [1.0, 1.0]),
    ([1.0, 0.0], [0.0], [5.0]),
])
def test_undamped_chain_on_a_pole_is_an_error(lib, alpha, beta, gamma):
    """Exactly singular matrices whose elimination from the top is exact."""
    tm = lib
    m = len(alpha)
    say(f"chi singular {alpha}")
    rng = np.random.default_rng(3)
    co = dict(alpha=np.array(alpha, complex), beta=np.array(beta + [1.0]), gamma=np.array(gamma + [1.0], complex),
              z=rng.standard_normal((3, m)) + 0j, zn=rng.standard_normal(m) + 0j, n1=1.0, steps_done=m)
    with pytest.raises(tm.TmError) as e:
        tm.tm_chi(co, m, np.array([0.375, 0.0]), 0.0)
    assert e.value.code == tm.TM_EINVAL
    assert np.isfinite(tm.tm_chi(co, m, np.array([0.375]), 0.0)).all()
