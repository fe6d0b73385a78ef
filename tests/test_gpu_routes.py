"""Which kernels a call runs, by the timing record: the autotuner's verdict and
an installed route decide between the launches and the persistent launch, in
both directions."""
import numpy as np
import pytest
import torch

from paper_2205_04295_amd import tune
from synth import workloads as wl

from gpu_util import need_gpu, rel_l2, run_gpu, run_oracle, to_dev

pytestmark = pytest.mark.gpu

EPIE = dict(alpha_obj=0.9, alpha_probe=0.9, beta=1.0, gamma=1.0)


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


def ran(call):
    """(result of call, kernels of the sweep that it launched)."""
    from paper_2205_04295_amd import api
    api.timing_enable(1)
    try:
        out = call()
        torch.cuda.synchronize()
        counts = api.timing_read()
    finally:
        api.timing_enable(0)
    return out, {k for k, v in counts.items() if v[1] > 0}


def batch(ws, **kw):
    from paper_2205_04295_amd import api
    jobs = [dict(obj=d["obj"], probe=d["probe"], pos=d["pos"], intens=d["I"],
                 err=torch.zeros(kw["iterations"], dtype=torch.float32, device="cuda:0"),
                 status=torch.zeros(1, dtype=torch.int32, device="cuda:0")) for d in map(to_dev, ws)]
    api.rpie_batched(jobs, **kw)
    return jobs


@pytest.mark.parametrize("N,M,jobs", [(64, 2, 1), (192, 3, 1), (256, 5, 2), (128, 1, 20)])
def test_autotuner_verdict_decides(N, M, jobs):
    cls = tune.call_class(jobs)
    saved = tune.get_tuning(N, cls, M=M)
    ws = [wl.small_case(900 + b, N + 19, N, M, 3, W=N + 26, name=f"a{b}") for b in range(jobs)]
    prm = dict(EPIE, iterations=1)
    try:
        best, times = tune.autotune(N, M, batch=jobs, J=8, reps=1)
        route = tune.get_route(N, cls, M=M)
        assert route in ("launches", "persistent")
        _, kernels = ran(lambda: batch(ws, **prm))
        team = route == "persistent" or (M <= best["lds_sweep"] and tune.lds_fits(N, M))
        print(N, M, jobs, route, best, sorted(kernels))
        assert ("k_team" in kernels) == team
    finally:
        tune.set_tuning(N, cls, M=M, **saved)
    assert tune.get_route(N, cls, M=M) == "auto"


@pytest.mark.parametrize("N,M", [(32, 3), (64, 1), (128, 2), (192, 3), (256, 3), (256, 5)])
def test_installed_route_decides(N, M):
    """... with the default tuning installed, whatever the library would choose."""
    w = wl.small_case(930, N + 19, N, M, 4, W=N + 26, name="r")
    prm = dict(EPIE, iterations=2)
    saved = tune.get_tuning(N, 0, M=M)
    tune.set_tuning(N, 0, M=M, **dict(saved, lds_sweep=0))  # (its lds_sweep would ask for the persistent launch)
    try:
        tune.set_route(N, 0, "launches", M=M)
        a, ka = ran(lambda: run_gpu(w, prm))
        tune.set_route(N, 0, "persistent", M=M)
        b, kb = ran(lambda: run_gpu(w, prm))
    finally:
        tune.set_tuning(N, 0, M=M, **saved)
    assert "k_rows" in ka and "k_team" not in ka
    assert "k_team" in kb and "k_rows" not in kb
    o = run_oracle(w, prm)
    for g in (a, b):
        assert rel_l2(g["O"], o["O"]) < 1e-4 and rel_l2(g["P"], o["P"]) < 1e-4 and g["status"] == 0
    assert rel_l2(a["O"], b["O"]) < 1e-5 and np.allclose(a["err"], b["err"], rtol=1e-5, atol=0)


@pytest.mark.parametrize("N,modes,J,want", [
    (192, (4, 5), (6, 6), {"k_rows"}), (192, (4,) * 7 + (5,), (6,) * 8, {"k_team"}),
    (192, (3, 3, 5, 5), (6,) * 4, {"k_rows"}), (256, (3, 5), (4, 4), {"k_rows"}),
    (256, (3, 8), (4, 4), {"k_rows"}), (256, (3,) * 7 + (8,), (3,) * 8, {"k_team", "k_rows"}),
    (256, (3, 3, 8), (4, 4, 1), {"k_team", "k_rows"})])
def test_jobs_of_a_call_run_one_way_together(N, modes, J, want):
    """Jobs of which some suit the persistent launch and some do not, and jobs
    that it does not hold: one route by most of the work, two only where few
    are left over."""
    ws = [wl.small_case(950 + b, N + 19, N, M, j, W=N + 26, name=f"t{b}") for b, (M, j) in enumerate(zip(modes, J))]
    prm = dict(EPIE, iterations=2)
    jobs, kernels = ran(lambda: batch(ws, **prm))
    assert kernels & {"k_team", "k_rows"} == want
    for j, w in zip(jobs, ws):
        o = run_oracle(w, prm)
        assert rel_l2(j["obj"].cpu().numpy(), o["O"]) < 1e-4
        assert rel_l2(j["probe"].cpu().numpy(), o["P"]) < 1e-4
        assert int(j["status"].item()) == 0
