"""The autotuner times the launches that applies and chains issue, and no others."""
import re

import pytest
import torch

from gpu_util import desc_from_problem, say
from test_gpu_planes import _problem
from test_gpu_tuning_order import _desc, _tuned

pytestmark = pytest.mark.gpu

PRODUCTS = re.compile(r"k_(gemm|cn_|reduce_pair|dmat|coefficients|update)")


def _kernels(tm):
    """Names of the profiled launches, without template arguments."""
    return {re.sub(r"<.*", "", name.strip("( ")) for name in tm.tm_profile_read()}


@pytest.mark.parametrize("nbnd", [7, 49])
def test_tuned_products_are_those_that_run(nbnd):
    """7 bands: one tile, both products in k_cn_pair; 49: the LDS-staged contraction."""
    import paper_2203_01120_amd as tm
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    tm.load()
    assert not _tuned(tm, nbnd), "another test already tuned this shape"
    h = tm.tm_system_create(_desc(tm, nbnd))
    try:
        say(f"launches of the tuner, 24^3, {nbnd} bands")
        n = tm.tm_qset_info_get(h, 0)["nelem"]
        x = torch.randn(n, dtype=torch.complex128, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
        y = torch.empty_like(x)
        tm.tm_profile_enable(True)
        tm.tm_profile_reset()
        tm.tm_liouvillian_apply(h, 0, x, y)
        tuning = _kernels(tm)
        tm.tm_profile_reset()
        tm.tm_liouvillian_apply(h, 0, x, y)
        tm.tm_chains_use_graphs(False)
        tm.tm_lanczos_run(h, 0, "z", "pH", 2)
        running = _kernels(tm)
        tm.tm_profile_enable(False)
        say(f"  tuner {sorted(tuning)}, after it {sorted(running)}")
        assert any(PRODUCTS.match(k) for k in running)
        assert {k for k in tuning if PRODUCTS.match(k)} <= running
        # the merged update has a choice of its own, between kernels with the same result
        entry = [e for e in _tuned(tm, nbnd) if e["op"] == "update_pair" and e["shape"].startswith("nonlocal")]
        assert len(entry) == 1 and entry[0]["variants"] == len(entry[0]["us"]) == 2
        for v in range(2):
            other = torch.empty_like(y)
            tm.tm_autotune_force("update_pair", v)
            tm.tm_liouvillian_apply(h, 0, x, other)
            torch.cuda.synchronize()
            assert torch.equal(other, y), v
    finally:
        tm.tm_autotune_force("update_pair", -1)
        tm.tm_chains_use_graphs(True)
        tm.tm_profile_enable(False)
        tm.tm_system_destroy(h)


@pytest.mark.parametrize("side,n3,r1,r2,variants", [(20, 6, 5, 4, 1), (24, 6, 9, 8, 1), (45, 5, 6, 7, 1), (48, 6, 18, 16, 2)])
def test_density_kernels_that_are_one_are_not_timed(side, n3, r1, r2, variants):
    """One variant on the matrix cores (fixed and other sides), two of the wave kernel."""
    import paper_2203_01120_amd as tm
    tm.load()
    prob = _problem(side, side, n3, r1, r2, 4, 37)
    h = tm.tm_system_create(desc_from_problem(prob))
    try:
        say(f"density variants, {side} x {side} x {n3}")
        n = tm.tm_qset_info_get(h, 0)["nelem"]
        x = torch.randn(n, dtype=torch.complex128, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
        y = torch.empty_like(x)
        tm.tm_liouvillian_apply(h, 0, x, y)
        entries = [e for e in tm.tm_autotune_report()
                   if e["op"] == "plane_density" and f"{side}x{side}x{n3}, 4 bands, 1 k" in e["shape"]]
        say(f"  {entries}")
        assert len(entries) == 1
        e = entries[0]
        assert e["variants"] == variants and len(e["us"]) == (variants if variants > 1 else 0)
        with pytest.raises(tm.TmError):
            tm.tm_autotune_force("plane_density", variants)
            tm.tm_liouvillian_apply(h, 0, x, y)
    finally:
        tm.tm_autotune_force("plane_density", -1)
        tm.tm_system_destroy(h)


def _tuned_apply_planes(tm, n1, n2, n3, r1, r2, nb, limit):
    """The plane_apply entries of a shape after a first apply of it."""
    h = tm.tm_system_create(desc_from_problem(_problem(n1, n2, n3, r1, r2, nb, 41)))
    try:
        say(f"plane tuning, {n1} x {n2} x {n3}, reach {r1}, {r2}, resident limit {limit}")
        tm.tm_system_set_resident_limit(h, limit)
        n = tm.tm_qset_info_get(h, 0)["nelem"]
        x = torch.randn(n, dtype=torch.complex128, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
        tm.tm_liouvillian_apply(h, 0, x, torch.empty_like(x))
        torch.cuda.synchronize()
        return [e for e in tm.tm_autotune_report()
                if e["op"] == "plane_apply" and f"{n1}x{n2}x{n3}, {nb} bands, 1 k" in e["shape"]]
    finally:
        tm.tm_system_destroy(h)


def test_spheres_of_other_kernels_are_tuned_by_themselves():
    """The reach of the spheres decides which matrix-core kernel runs."""
    import paper_2203_01120_amd as tm
    tm.load()
    assert len(_tuned_apply_planes(tm, 20, 20, 6, 5, 4, 7, -1)) == 1
    assert len(_tuned_apply_planes(tm, 20, 20, 6, 5, 4, 7, -1)) == 1     # known by now
    assert len(_tuned_apply_planes(tm, 20, 20, 6, 9, 6, 7, -1)) == 2


def test_wave_and_matrix_core_kernels_are_tuned_by_themselves():
    """48 planes by columns on the matrix cores, and 96 with the resident ground
    state of full spheres on the wave kernels."""
    import paper_2203_01120_amd as tm
    tm.load()
    assert len(_tuned_apply_planes(tm, 48, 48, 48, 12, 10, 7, 0)) == 1
    assert len(_tuned_apply_planes(tm, 48, 48, 96, 18, 16, 7, -1)) == 1
