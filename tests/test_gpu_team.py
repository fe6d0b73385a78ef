"""The persistent sweep (teams of workgroups on one XCD) against the row /
column passes and the oracle: every probe size and mode count it takes, team
sizes 32, 16, 8 and 4 by the number of jobs, more jobs than teams, one
position, ragged objects, mixed sizes in one launch.

Both paths run fp32 FFTs with fp32 sums over the modes; their roundings
differ by a few ulp (6e-8) in each of a handful of updates, so 1e-5 against
the passes and 1e-4 against the fp64 oracle, as in the tests of the passes.
The updates are M-ePIE's: the rPIE weights divide by the
local intensity, which amplifies rounding where a small probe is dark."""
import numpy as np
import pytest
import torch

from paper_2205_04295_amd import tune
from synth import workloads as wl

from gpu_util import need_gpu, rel_l2, run_gpu, run_oracle, to_dev, tuning

pytestmark = pytest.mark.gpu

EPIE = dict(alpha_obj=0.9, alpha_probe=0.9, beta=1.0, gamma=1.0)


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


def run_jobs(ws, prm):
    from paper_2205_04295_amd import api
    devs = [to_dev(w) for w in ws]
    jobs = [dict(obj=d["obj"], probe=d["probe"], pos=d["pos"], intens=d["I"],
                 err=torch.zeros(prm["iterations"], dtype=torch.float32, device="cuda:0"),
                 status=torch.zeros(1, dtype=torch.int32, device="cuda:0")) for d in devs]
    api.rpie_batched(jobs, **prm)
    torch.cuda.synchronize()
    return [dict(O=j["obj"].cpu().numpy(), P=j["probe"].cpu().numpy(), err=j["err"].cpu().numpy(),
                 status=int(j["status"].item())) for j in jobs]


def close(a, b):
    assert rel_l2(a["O"], b["O"]) < 1e-5
    assert rel_l2(a["P"], b["P"]) < 1e-5
    assert np.allclose(a["err"], b["err"], rtol=1e-5, atol=0)
    assert a["status"] == b["status"]


@pytest.mark.parametrize("N,M,jobs,J", [
    (32, 1, 1, 1), (32, 8, 1, 5), (32, 3, 9, 5), (32, 2, 65, 3),
    (64, 1, 17, 4), (64, 5, 1, 4), (64, 8, 33, 3), (64, 3, 70, 3),
    (128, 1, 33, 3), (128, 4, 1, 4), (128, 6, 9, 3), (128, 8, 17, 3),
    (192, 1, 2, 3), (192, 4, 8, 3), (192, 3, 3, 3),
    (256, 1, 17, 3), (256, 2, 9, 3), (256, 3, 1, 4), (256, 3, 18, 3), (256, 4, 1, 3), (256, 6, 3, 3)])
def test_team_matches_passes_and_oracle(N, M, jobs, J):
    ws = [wl.small_case(500 + b % 3, N + 17 + 2 * (b % 3), N, M, J, W=N + 30 - b % 3, name=f"t{b % 3}") for b in range(jobs)]
    prm = dict(EPIE, iterations=2)
    got = run_jobs(ws, prm)
    with tuning(N, tune.call_class(jobs), cols_radix=4, lds_sweep=0):   # an installed setting: the passes
        ref = [run_gpu(ws[0], prm)] if jobs == 1 else run_jobs(ws, prm)
    for a, b in zip(got, ref):
        close(a, b)
    o = run_oracle(ws[0], prm)
    assert rel_l2(got[0]["O"], o["O"]) < 1e-4
    assert rel_l2(got[0]["P"], o["P"]) < 1e-4


def test_team_mixed_sizes_clamp_and_start():
    """One launch of every size; positions off the object are clamped and
    flagged; probe updates that start late."""
    specs = [(32, 3), (64, 2), (128, 5), (192, 1), (256, 3), (256, 1), (64, 8), (32, 1), (128, 2), (192, 2)]
    ws = [wl.small_case(600 + i, N + 25, N, M, 4 + i % 3, W=N + 12, name=f"m{i}") for i, (N, M) in enumerate(specs)]
    ws[2].pos0[3] = (400.0, -3.0)
    for extra in (dict(), dict(probe_update_start=1)):
        prm = dict(EPIE, iterations=2, **extra)
        got = run_jobs(ws, prm)
        assert [g["status"] != 0 for g in got] == [i == 2 for i in range(len(ws))]
        with tuning(256, tune.call_class(len(ws)), cols_radix=4):
            for a, b in zip(got, run_jobs(ws, prm)):
                close(a, b)


def test_long_call_is_cut_at_iterations():
    """More positions than one launch takes (65536 of a team): the launches
    resume with the same bits as calls of the caller's own."""
    from paper_2205_04295_amd import api
    w = wl.small_case(700, 48, 32, 1, 5, name="long")
    T = 14000
    one = run_gpu(w, dict(EPIE, iterations=T))
    d = to_dev(w)
    err = torch.zeros(T, dtype=torch.float32, device="cuda:0")
    for it in range(0, T, 7000):
        api.rpie(d["obj"], d["probe"], d["pos"], d["I"], err=err[it:], iter_offset=it,
                 **dict(EPIE, iterations=7000))
    torch.cuda.synchronize()
    assert np.array_equal(one["O"], d["obj"].cpu().numpy())
    assert np.array_equal(one["P"], d["probe"].cpu().numpy())
    assert np.array_equal(one["err"], err.cpu().numpy()) and (one["err"] > 0).all()
