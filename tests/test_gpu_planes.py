"""Plane kernels at the edges of their tiles, against the oracle (needs an MI355X).

Cells are boxes whose sides set the reach |m1|, |m2| of the plane-wave spheres,
so that every K-step count, row and column remainder and dispatch line is met:
the fixed plane sizes with half-filled and full spheres, the fullest ones on
the radix kernels, odd and unequal sides, the largest plane, and planes that
the matrix-core kernels do not take.

Tolerance: FP64 with different summation orders only, 1e-12 relative as for
the other apply tests; right-hand sides in one pass equal single applies, and
the lanes of a chain single chains, bit for bit.
"""
import numpy as np
import pytest

import synth
from oracle import liouvillian as lv

from gpu_util import desc_from_problem, from_gpu, rel_err, say, to_gpu

pytestmark = pytest.mark.gpu

# n1, n2, n3, reach along i1 and i2
PLANES = [
    (8, 8, 8, 3, 2), (20, 20, 20, 5, 4), (20, 20, 6, 9, 6), (24, 24, 6, 7, 7), (24, 24, 6, 8, 11),
    (32, 32, 6, 8, 8), (32, 32, 6, 12, 15), (48, 48, 6, 11, 11), (48, 48, 6, 10, 13), (48, 48, 6, 14, 9),
    (48, 48, 5, 23, 20),
    (4, 5, 6, 1, 2), (5, 4, 5, 2, 1), (9, 15, 6, 4, 7), (16, 10, 9, 7, 4), (27, 25, 5, 12, 8),
    (30, 32, 6, 11, 15), (36, 50, 6, 3, 20), (45, 40, 5, 19, 16), (40, 45, 5, 12, 22), (60, 64, 5, 16, 15),
    (64, 64, 5, 11, 17), (64, 8, 6, 23, 3), (3, 8, 6, 1, 3), (72, 6, 6, 7, 2), (64, 64, 5, 23, 23),
]


def _problem(n1, n2, n3, r1, r2, nb, seed):
    base = synth.make_tiny(nbnd=nb, seed=seed)
    ecut = 2.0   # |k + G| <= 2: a side of pi (r + 0.3) holds |m| <= r for |q| <= 0.2 of a cell
    cell = np.diag([np.pi * (r + 0.3) for r in (r1, r2, 1)])
    sd = synth.SystemDef(name="box", cell=cell, atoms=base.atoms, ecut=ecut, fft=(n1, n2, n3), nbnd=nb,
                         kmesh=np.zeros((1, 3)), seed=seed)
    inp = synth.synthetic_inputs(sd, synth.cart_from_frac(sd, [0.1, 0.05, 0.0]), seed=seed)

    class _GS:
        pass
    gs = _GS()
    gs.sysd, gs.vrs, gs.rho = inp["sysd"], inp["vrs"], inp["rho"]
    prob = lv.Problem(gs, inp["qset"], point_states=[(m, e, et) for (_, m, e, et, _) in inp["points"]])
    reach = np.max([np.abs(m).max(axis=0) for (_, m, _, _, _) in inp["points"]], axis=0)
    assert tuple(reach[:2]) == (r1, r2), reach
    return prob


@pytest.mark.parametrize("n1,n2,n3,r1,r2", PLANES)
def test_apply_at_tile_edges(n1, n2, n3, r1, r2):
    import torch
    import paper_2203_01120_amd as tm
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    prob = _problem(n1, n2, n3, r1, r2, 5, 17)
    h = tm.tm_system_create(desc_from_problem(prob))
    try:
        info = tm.tm_qset_info_get(h, 0)
        shape = (2, 1, prob.nb, 2, info["npw_pad"])
        nrhs = 3
        xs = [prob.random_projected(seed) for seed in (1, 2)]
        refs = [prob.apply(x) for x in xs]
        xin = torch.cat([to_gpu(xs[i % 2], info["npw_pad"]) for i in range(nrhs)])
        n = xin.numel() // nrhs
        for limit in (-1, 0):   # resident ground state (where the plane size has it), columns
            tm.tm_system_set_resident_limit(h, limit)
            say(f"plane {n1} x {n2}, reach {r1}, {r2}, resident limit {limit}")
            single = torch.empty_like(xin[:2 * n])
            for i in range(2):
                tm.tm_liouvillian_apply(h, 0, xin[i * n:(i + 1) * n], single[i * n:(i + 1) * n])
            out = torch.empty_like(xin)
            tm.tm_liouvillian_apply_multi(h, 0, nrhs, xin, out)
            torch.cuda.synchronize()
            for i in range(2):
                got, raw = from_gpu(single[i * n:(i + 1) * n], shape, prob.npw_pad)
                assert rel_err(got, refs[i]) <= 1e-12, rel_err(got, refs[i])
                assert np.all(raw[:, 0, :, :, prob.k[0].npw:] == 0)
            for i in range(nrhs):
                assert torch.equal(out[i * n:(i + 1) * n], single[i % 2 * n:(i % 2 + 1) * n])
    finally:
        tm.tm_system_destroy(h)


def test_many_lanes_equal_single_chains():
    """15 lanes at 20^3 are enough blocks for each to hold all bands of a side,
    whose chunks' sums then add up in the block instead of in the reduction."""
    import paper_2203_01120_amd as tm
    prob = _problem(20, 20, 20, 5, 4, 9, 23)
    h = tm.tm_system_create(desc_from_problem(prob))
    try:
        say("plane 20 x 20, 15 lanes")
        dirs = ["+", "-", "z"] * 5
        chain = tm.tm_chain_begin_lanes(h, [0] * 15, dirs, "pH", 4)
        try:
            tm.tm_chains_step([chain], 4)
            lanes = tm.tm_chain_coeffs_lanes(chain, 4)
        finally:
            tm.tm_chain_end(chain)
        for i, d in enumerate(dirs[:3]):
            one = tm.tm_lanczos_run(h, 0, d, "pH", 4)
            for key in ("alpha", "beta", "gamma", "z"):
                for lane in lanes[i::3]:
                    assert np.array_equal(lane[key], one[key]), (d, key)
    finally:
        tm.tm_system_destroy(h)


@pytest.mark.parametrize("n1,n2,n3", [(8, 8, 16), (8, 16, 9), (10, 9, 125), (6, 5, 300), (64, 64, 24), (128, 30, 6),
                                      (24, 24, 20), (32, 32, 32), (20, 20, 25)])
def test_potential_at_its_limits(n1, n2, n3):
    """The response potential where its launches change: the largest grid of one
    block and the first past it, the longest columns in LDS and the first too
    long, 16 columns a block, the largest and a long plane, and the compile-time
    plane and column lengths apart and together; an apply to 1e-12 as above."""
    import torch
    import paper_2203_01120_amd as tm
    prob = _problem(n1, n2, n3, 2, 2, 3, 29)
    h = tm.tm_system_create(desc_from_problem(prob))
    try:
        say(f"potential {n1} x {n2} x {n3}")
        info = tm.tm_qset_info_get(h, 0)
        x = prob.random_projected(1)
        xin = to_gpu(x, info["npw_pad"])
        out = torch.empty_like(xin)
        tm.tm_liouvillian_apply(h, 0, xin, out)
        torch.cuda.synchronize()
        got, _ = from_gpu(out, (2, 1, prob.nb, 2, info["npw_pad"]), prob.npw_pad)
        err = rel_err(got, prob.apply(x))
        assert err <= 1e-12, err
    finally:
        tm.tm_system_destroy(h)
