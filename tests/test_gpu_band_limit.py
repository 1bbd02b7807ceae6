"""The band limit of the nonlocal term's update, 256 columns (both spins of a
band), holds whether or not the autotuner has run and in both precisions."""
import pytest

from paper_2203_01120_amd.binding import TM_EUNSUPPORTED

from gpu_util import desc_from_problem, from_gpu, rel_err, say, to_gpu
from test_gpu_planes import _problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb", [128, 129])
def test_projectors_of_more_than_128_bands_are_refused(nb):
    import torch
    import paper_2203_01120_amd as tm
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    prob = _problem(24, 24, 8, 8, 8, nb, 31)
    h = tm.tm_system_create(desc_from_problem(prob))
    tm.tm_autotune_enable(False)
    try:
        say(f"{nb} bands with projectors")
        info = tm.tm_qset_info_get(h, 0)
        x = prob.random_projected(1)
        xin = to_gpu(x, info["npw_pad"])
        out = torch.empty_like(xin)
        if nb <= 128:
            tm.tm_liouvillian_apply(h, 0, xin, out)
            torch.cuda.synchronize()
            got, _ = from_gpu(out, (2, 1, prob.nb, 2, info["npw_pad"]), prob.npw_pad)
            err = rel_err(got, prob.apply(x))
            assert err <= 1e-12, err
            return
        for prec in (tm.TM_FP64, tm.TM_FP32):
            with pytest.raises(tm.TmError) as e:
                tm.tm_liouvillian_apply(h, 0, xin, out, prec)
            assert e.value.code == TM_EUNSUPPORTED
    finally:
        tm.tm_autotune_enable(True)
        tm.tm_system_destroy(h)
