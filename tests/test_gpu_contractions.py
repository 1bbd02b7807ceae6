"""The nonlocal term and the projector together, at the edges of their tiles and
routes, against the oracle (needs an MI355X): one band; a full tile and one more;
the last band count with in-register tiles and the first staged through LDS;
projectors in one tile and in two; partial sums added up by the coefficient
kernel or in a launch of their own.

Tolerance: FP64 with different summation orders only, 1e-12 relative; right-hand
sides in one pass equal single applies bit for bit.
"""
import dataclasses

import numpy as np
import pytest

import synth
from oracle import liouvillian as lv

from gpu_util import desc_from_problem, from_gpu, rel_err, say, to_gpu

pytestmark = pytest.mark.gpu


def _problem(nb, nat, mesh):
    base = synth.make_tiny(nbnd=nb, seed=31)
    rng = np.random.default_rng(nat)
    atoms = [dataclasses.replace(base.atoms[i % 2], pos=rng.uniform(0.0, 8.0, 3)) for i in range(nat)]
    f = np.arange(mesh) / mesh
    sd = synth.SystemDef(name="box", cell=np.diag([9.0, 8.0, 10.0]), atoms=atoms, ecut=2.0, fft=(15, 12, 16), nbnd=nb,
                         kmesh=np.array([[a, 0.0, 0.0] for a in f]), seed=31)
    inp = synth.synthetic_inputs(sd, synth.cart_from_frac(sd, [0.1, 0.05, 0.0]), seed=31)

    class _GS:
        pass
    gs = _GS()
    gs.sysd, gs.vrs, gs.rho = inp["sysd"], inp["vrs"], inp["rho"]
    return lv.Problem(gs, inp["qset"], point_states=[(m, e, et) for (_, m, e, et, _) in inp["points"]])


@pytest.mark.parametrize("nb,nat,mesh", [(1, 1, 1), (16, 2, 1), (17, 8, 2), (32, 9, 1), (33, 9, 1), (48, 2, 3), (3, 20, 1)])
def test_nonlocal_and_projector_match_oracle(nb, nat, mesh):
    import torch
    import paper_2203_01120_amd as tm
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    prob = _problem(nb, nat, mesh)
    h = tm.tm_system_create(desc_from_problem(prob))
    try:
        say(f"contractions {nb} bands, {nat} atoms, {mesh} k")
        info = tm.tm_qset_info_get(h, 0)
        xs = [prob.random_projected(seed) for seed in (1, 2)]
        xin = torch.cat([to_gpu(xs[i % 2], info["npw_pad"]) for i in range(3)])
        n = xin.numel() // 3
        out, single = torch.empty_like(xin), torch.empty_like(xin[:n])
        tm.tm_liouvillian_apply_multi(h, 0, 3, xin, out)
        for i in range(2):
            tm.tm_liouvillian_apply(h, 0, xin[i * n:(i + 1) * n], single)
            torch.cuda.synchronize()
            assert torch.equal(out[i * n:(i + 1) * n], single)
            got, _ = from_gpu(single, (2, mesh, nb, 2, info["npw_pad"]), prob.npw_pad)
            err = rel_err(got, prob.apply(xs[i]))
            assert err <= 1e-12, err
        assert torch.equal(out[2 * n:], out[:n])
    finally:
        tm.tm_system_destroy(h)
