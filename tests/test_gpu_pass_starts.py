"""A single sweep's row and column passes give the same results however their
workgroups happen to start: timing the launches spreads the starts, and every
timed call's outputs are the untimed call's (float rounding between two runs,
rel L2 1e-5).  The passes exchange spectra in two layouts, which must not share
a buffer."""
import numpy as np
import pytest
import torch

from paper_2205_04295_amd import api, tune
from synth import workloads as wl

from gpu_util import need_gpu, rel_l2, to_dev

pytestmark = pytest.mark.gpu

EPIE = dict(alpha_obj=0.9, alpha_probe=0.9, beta=1.0, gamma=1.0, iterations=2)


@pytest.mark.parametrize("N,M", [(32, 1), (64, 1), (128, 2)])
def test_spread_starts_do_not_change_the_passes(N, M):
    need_gpu()
    w = wl.small_case(930, N + 19, N, M, 4, W=N + 26, name="t")
    passes = dict(tune.get_tuning(N, 0, M=M), lds_sweep=0)

    def sweep(stride):
        d = to_dev(w)
        err = torch.zeros(2, dtype=torch.float32, device="cuda:0")
        job = dict(obj=d["obj"], probe=d["probe"], pos=d["pos"], intens=d["I"], err=err)
        api.timing_enable(stride)
        try:
            api.rpie_batched([job], tuning=passes, **EPIE)
            torch.cuda.synchronize()
            n = api.timing_read()["k_rows"][1]
        finally:
            api.timing_enable(0)
        assert (n > 0) == (stride > 0)
        return d["obj"].cpu().numpy(), err.cpu().numpy()

    obj, err = sweep(0)
    wrong = 0
    for stride in [1, 1, 0, 2, 0] * 60:
        o, e = sweep(stride)
        wrong += not (rel_l2(o, obj) < 1e-5 and np.allclose(e, err, rtol=1e-5, atol=0))
    assert wrong == 0
