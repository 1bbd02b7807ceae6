"""Each route of the response potential, told by the launches of an apply: one
block for the whole grid, planes and columns in LDS, and line transforms of the
whole grid where a column is too long for a block.

Columns of n3 points fit with 8 n3 / r <= 1024 butterflies (r: the smallest
radix among 4, 5, 3, 2 that divide n3 in turn): 250 (r = 2), 300 (3) and 256 (4)
do, 270 (2) does not.  Planes of 4096 points take 16 columns a block for
lengths without a kernel of their own.

Tolerance: FP64 in another order of summation, 1e-12 relative; three
right-hand sides in one pass equal single applies bit for bit.
"""
import pytest
import torch

from gpu_util import desc_from_problem, from_gpu, rel_err, say, to_gpu
from test_gpu_planes import _problem

pytestmark = pytest.mark.gpu

LINES = {"k_copy_scale", "k_mul_real", "k_assemble_W"}
PLANES = {"k_rho_planes", "k_pot_columns", "k_pot_planes"}
BLOCK = {"k_potential_lds"}


@pytest.mark.parametrize("n1,n2,n3,route", [
    (8, 16, 8, BLOCK), (8, 16, 9, PLANES),
    (6, 5, 250, PLANES), (6, 5, 300, PLANES), (5, 6, 256, PLANES), (64, 64, 25, PLANES), (64, 64, 30, PLANES),
    (6, 5, 270, LINES),       # matrix-core planes of even and odd sides
    (9, 10, 270, LINES),
    (8, 8, 270, LINES),       # with the resident ground state
    (3, 8, 270, LINES),       # generic plane kernels
    (3, 8, 9, BLOCK), (3, 8, 45, PLANES),
])
def test_potential_route(n1, n2, n3, route):
    import paper_2203_01120_amd as tm
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    small = min(n1, n2) < 5
    prob = _problem(n1, n2, n3, 1 if small else 2, 2, 3, 29)
    h = tm.tm_system_create(desc_from_problem(prob))
    try:
        say(f"potential {n1} x {n2} x {n3}: {sorted(route)}")
        info = tm.tm_qset_info_get(h, 0)
        xs = [prob.random_projected(seed) for seed in (1, 2)]
        xin = torch.cat([to_gpu(xs[i % 2], info["npw_pad"]) for i in range(3)])
        n = xin.numel() // 3
        single = torch.empty_like(xin[:2 * n])
        for i in range(2):
            tm.tm_liouvillian_apply(h, 0, xin[i * n:(i + 1) * n], single[i * n:(i + 1) * n])
        out = torch.empty_like(xin)
        tm.tm_profile_enable(True)
        tm.tm_profile_reset()
        tm.tm_liouvillian_apply_multi(h, 0, 3, xin, out)
        torch.cuda.synchronize()
        ran = {k.split("<")[0].strip("( ") for k in tm.tm_profile_read()}
        assert route <= ran and not (LINES | PLANES | BLOCK) - route & ran, ran
        for i in range(2):
            got, _ = from_gpu(single[i * n:(i + 1) * n], (2, 1, prob.nb, 2, info["npw_pad"]), prob.npw_pad)
            err = rel_err(got, prob.apply(xs[i]))
            assert err <= 1e-12, err
        for i in range(3):
            assert torch.equal(out[i * n:(i + 1) * n], single[i % 2 * n:(i % 2 + 1) * n])
    finally:
        tm.tm_profile_enable(False)
        tm.tm_system_destroy(h)
