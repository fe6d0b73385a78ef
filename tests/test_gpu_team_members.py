"""Persistent sweep in teams with too few workgroups for their job's units (what
a launch forms when it finds the GPU busy): every wave takes its units in
turn.  Sums are taken in the full teams' order, so the results are theirs bit
for bit; the oracle's to the sweep's tolerance (rel L2 1e-4, M-ePIE weights as
in the tests of full teams)."""
import numpy as np
import pytest
import torch

from synth import workloads as wl

from gpu_util import need_gpu, rel_l2, run_oracle, to_dev

pytestmark = pytest.mark.gpu

EPIE = dict(alpha_obj=0.9, alpha_probe=0.9, beta=1.0, gamma=1.0)


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


def team(ws, members, wait_ns=0, **prm):
    from paper_2205_04295_amd import api
    devs = [to_dev(w) for w in ws]
    jobs = [dict(obj=d["obj"], probe=d["probe"], pos=d["pos"], intens=d["I"],
                 err=torch.zeros(prm["iterations"], dtype=torch.float32, device="cuda:0"),
                 status=torch.zeros(1, dtype=torch.int32, device="cuda:0")) for d in devs]
    api.team_sweep(jobs, members=members, wait_ns=wait_ns, **prm)
    torch.cuda.synchronize()
    return [dict(O=j["obj"].cpu().numpy(), P=j["probe"].cpu().numpy(), err=j["err"].cpu().numpy(),
                 status=int(j["status"].item())) for j in jobs]


def check(ws, members, prm):
    for weights in (dict(beta=0.6, gamma=0.3), dict()):
        full = team(ws, 32, **dict(prm, **weights))
        got = team(ws, members, **dict(prm, **weights))
        for a, b in zip(got, full):
            assert np.array_equal(a["O"], b["O"]) and np.array_equal(a["P"], b["P"])
            assert np.array_equal(a["err"], b["err"]) and a["status"] == b["status"]
    o = run_oracle(ws[0], prm)
    assert rel_l2(got[0]["O"], o["O"]) < 1e-4
    assert rel_l2(got[0]["P"], o["P"]) < 1e-4


# a team of one, odd sizes, one member short; mode counts that leave some
# waves a mode less (5 of 192^2 in twos, 5 of 256^2 in threes); several jobs a team
@pytest.mark.parametrize("N,M,jobs,J,members", [
    (32, 8, 1, 5, 1), (32, 3, 33, 3, 1), (64, 1, 1, 4, 3), (64, 5, 1, 4, 3), (64, 7, 33, 3, 3), (128, 2, 1, 3, 1),
    (128, 3, 9, 3, 10), (128, 7, 17, 2, 10), (192, 1, 2, 3, 10), (192, 5, 1, 3, 10), (256, 1, 1, 3, 10),
    (256, 3, 1, 3, 31), (256, 3, 9, 3, 10), (256, 4, 1, 2, 3), (256, 5, 1, 2, 10), (256, 3, 1, 2, 1)])
def test_small_teams_match_full_ones(N, M, jobs, J, members):
    ws = [wl.small_case(800 + b % 2, N + 19, N, M, J, W=N + 26, name=f"s{b % 2}") for b in range(jobs)]
    check(ws, members, dict(EPIE, iterations=2))


@pytest.mark.parametrize("members", [1, 3, 10])
def test_small_teams_of_mixed_sizes(members):
    specs = [(128, 3), (64, 2), (256, 3), (192, 3), (32, 5), (256, 1), (64, 8), (128, 5), (192, 2), (32, 1)]
    ws = [wl.small_case(820 + i, N + 21, N, M, 3 + i % 2, W=N + 12, name=f"x{i}") for i, (N, M) in enumerate(specs)]
    ws[3].pos0[1] = (999.0, -4.0)  # clamped and flagged in both
    check(ws, members, dict(EPIE, iterations=2, probe_update_start=1))


@pytest.mark.parametrize("N,M,jobs,members", [(256, 3, 3, 32), (128, 2, 20, 32), (64, 2, 1, 32), (256, 1, 12, 5)])
def test_wait_that_gives_up(N, M, jobs, members):
    """Waits inside a job that give up at once: the launch ends, a
    job is either swept as ever or flagged as unfinished, whichever member
    gave up and whoever had no part in it, and the next call is unharmed."""
    ws = [wl.small_case(860 + b % 2, N + 19, N, M, 60, W=N + 26, name=f"w{b % 2}") for b in range(jobs)]
    prm = dict(EPIE, iterations=2)
    ref = team(ws, members, **prm)
    got = team(ws, members, wait_ns=1, **prm)
    print([g["status"] for g in got])
    assert any(g["status"] == 4 for g in got)
    for a, b in zip(got, ref):
        assert a["status"] == 4 or (a["status"] == 0 and np.array_equal(a["O"], b["O"]))
    for a, b in zip(team(ws, members, **prm), ref):
        assert a["status"] == 0 and np.array_equal(a["O"], b["O"]) and np.array_equal(a["P"], b["P"])


def test_single_32_is_one_workgroup():
    """32^2 x 1 alone runs as a team of one; more jobs, and more modes, by two
    members each: the same bits."""
    from paper_2205_04295_amd import api
    for M in (1, 2):
        w = wl.small_case(880, 71, 32, M, 40, W=60, name="u")
        prm = dict(EPIE, iterations=3)
        many = team([w] * 9, 32, **prm)
        one = team([w], 32, **prm)[0]
        for members in (1, 2):
            g = team([w], members, **prm)[0]
            assert np.array_equal(g["O"], one["O"]) and np.array_equal(g["P"], one["P"])
            assert np.array_equal(g["err"], one["err"])
        for g in many:
            assert np.array_equal(g["O"], one["O"]) and np.array_equal(g["err"], one["err"])
        d = to_dev(w)
        api.rpie(d["obj"], d["probe"], d["pos"], d["I"], **prm)
        torch.cuda.synchronize()
        assert np.array_equal(d["obj"].cpu().numpy(), one["O"])
