"""The lock-step launches of batches and the row / column passes of single
sweeps, asked for by the call's tuning or the installed route (most calls of
these sizes would run the persistent launch), and the batches of 192^2 probes
that take them by default.  Tolerances as for the plain sweep: float rounding
between two ways (rel L2 1e-5), 1e-4 to the oracle."""
import threading

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


def make(ws, T):
    return [dict(obj=d["obj"], probe=d["probe"], pos=d["pos"], intens=d["I"],
                 err=torch.zeros(T, dtype=torch.float32, device="cuda:0"),
                 status=torch.zeros(1, dtype=torch.int32, device="cuda:0")) for d in map(to_dev, ws)]


def kernels_of(call):
    """Kernels of the sweep that `call` launches, by the timing record."""
    from paper_2205_04295_amd import api
    api.timing_enable(1)
    try:
        call()
        torch.cuda.synchronize()
        counts = api.timing_read()
    finally:
        api.timing_enable(0)
    return {k for k, v in counts.items() if v[1] > 0 and k in ("k_rows", "k_cols", "k_upd", "k_gat", "k_team")}


def default_shape(N, jobs, M):
    return dict(tune.get_tuning(N, tune.call_class(jobs), M=M), lds_sweep=0)


def alone(w, prm):
    """The job's own sweep as launches."""
    N, M = w.P0.shape[-1], w.P0.shape[0]
    saved = tune.get_tuning(N, 0, M=M)
    tune.set_tuning(N, 0, M=M, **dict(saved, lds_sweep=0))
    tune.set_route(N, 0, "launches", M=M)
    try:
        return run_gpu(w, prm)
    finally:
        tune.set_tuning(N, 0, M=M, **saved)


def check_against_alone(jobs, ws, prm):
    for j, w in zip(jobs, ws):
        g = alone(w, prm)
        assert rel_l2(j["obj"].cpu().numpy(), g["O"]) < 1e-5
        assert rel_l2(j["probe"].cpu().numpy(), g["P"]) < 1e-5
        assert np.allclose(j["err"].cpu().numpy(), g["err"], rtol=1e-5, atol=0)
        assert int(j["status"].item()) == 0


def check_oracle(j, w, prm):
    o = run_oracle(w, prm)
    assert rel_l2(j["obj"].cpu().numpy(), o["O"]) < 1e-4
    assert rel_l2(j["probe"].cpu().numpy(), o["P"]) < 1e-4


SPLIT, FUSED = {"k_upd", "k_gat", "k_cols"}, {"k_rows", "k_cols"}


def test_equal_jobs_on_more_lanes_than_a_launch_has():
    """80 jobs, 40 a stream: 4 of each stream wait for a lane."""
    from paper_2205_04295_amd import api
    w = wl.small_case(81, 96, 64, 1, 4, name="many")
    prm = dict(EPIE, iterations=1)
    jobs = make([w] * 80, 1)
    k = kernels_of(lambda: api.rpie_batched(jobs, tuning=default_shape(64, 80, 1), **prm))
    assert k == SPLIT
    for j in jobs[1:]:
        assert torch.equal(j["obj"], jobs[0]["obj"]) and torch.equal(j["probe"], jobs[0]["probe"])
    check_against_alone(jobs[:1], [w], prm)
    check_oracle(jobs[0], w, prm)


@pytest.mark.parametrize("capture", [False, True])
def test_ragged_jobs_on_more_lanes_than_a_launch_has(capture):
    """76 jobs of uneven sizes and scan lengths, eager on two streams and
    captured on one; every replay against the eager call."""
    from paper_2205_04295_amd import api, graph
    specs = [dict(seed=150 + i, H=(64, 64, 128, 128)[i % 4] + 40, N=(64, 64, 128, 128)[i % 4], M=1 + (i // 4) % 3,
                  J=2 + (5 * i) % 11) for i in range(76)]
    ws = [wl.small_case(name=f"l{i}", **s) for i, s in enumerate(specs)]
    prm = dict(EPIE, iterations=1)
    t = default_shape(128, 76, 3)
    eager = make(ws, 1)
    k = kernels_of(lambda: api.rpie_batched(eager, tuning=t, **prm))
    assert k == SPLIT
    check_against_alone(eager[::5], ws[::5], prm)
    if not capture:
        return
    jobs = make(ws, 1)
    g = graph.capture_batched(jobs, tuning=t, **prm)
    for rep in range(3):
        g.replay()
        if rep:
            api.rpie_batched(eager, tuning=t, **prm)
        torch.cuda.synchronize()
        for a, b in zip(jobs, eager):
            assert torch.equal(a["obj"], b["obj"]) and torch.equal(a["probe"], b["probe"]), rep
            assert torch.equal(a["err"], b["err"]), rep


def test_many_jobs_in_place():
    from paper_2205_04295_amd import api
    specs = [dict(seed=90 + i, H=192 if i % 2 else 256, N=128, M=1 + i % 3, J=3 + i % 4) for i in range(18)]
    ws = [wl.small_case(name=f"m{i}", **s) for i, s in enumerate(specs)]
    prm = dict(EPIE, iterations=2)
    jobs = make(ws, 2)
    t = default_shape(128, 18, 3)
    assert t["rows_inplace"] and t["cols_width"] == 4
    assert kernels_of(lambda: api.rpie_batched(jobs, tuning=t, **prm)) == SPLIT
    check_against_alone(jobs, ws, prm)
    check_oracle(jobs[4], ws[4], prm)


def test_large_probes_in_place_columns_many_modes():
    from paper_2205_04295_amd import api
    specs = [dict(seed=110 + i, H=(192, 256)[i % 2] + 64, N=(192, 256)[i % 2], M=(1, 3, 5)[i % 3], J=3 + i % 3)
             for i in range(16)]
    ws = [wl.small_case(name=f"w{i}", **s) for i, s in enumerate(specs)]
    prm = dict(EPIE, iterations=2)
    jobs = make(ws, 2)
    assert kernels_of(lambda: api.rpie_batched(jobs, tuning=default_shape(256, 16, 5), **prm)) == SPLIT
    check_against_alone(jobs, ws, prm)
    check_oracle(jobs[5], ws[5], prm)  # 256^2 x 5 modes


@pytest.mark.parametrize("inplace,width,split", [(1, 4, 0), (0, 1, 1)])
def test_fused_and_split_of_mixed_sizes(inplace, width, split):
    """(1, 4, 0) is the default shape of 2 to 15 jobs."""
    from paper_2205_04295_amd import api
    specs = [dict(seed=71, H=160, N=64, M=1, J=9), dict(seed=72, H=256, N=128, M=3, J=5),
             dict(seed=73, H=320, N=192, M=2, J=3), dict(seed=74, H=384, N=256, M=4, J=4),
             dict(seed=75, H=128, N=64, M=5, J=12), dict(seed=76, H=96, N=32, M=2, J=7)]
    ws = [wl.small_case(name=f"b{i}", **s) for i, s in enumerate(specs)]
    prm = dict(EPIE, iterations=2)
    jobs = make(ws, 2)
    t = dict(default_shape(256, 5, 4), rows_inplace=inplace, cols_width=width, rows_split=split)
    assert kernels_of(lambda: api.rpie_batched(jobs, tuning=t, **prm)) == (SPLIT if split else FUSED)
    check_against_alone(jobs, ws, prm)
    check_oracle(jobs[1], ws[1], prm)


def test_two_host_threads_fork_the_side_stream():
    """Every job ends bitwise equal to the same call made alone."""
    from paper_2205_04295_amd import api
    specs = [dict(seed=91, H=256, N=128, M=2, J=6), dict(seed=92, H=192, N=64, M=3, J=8),
             dict(seed=93, H=320, N=128, M=1, J=5)]
    ws = [wl.small_case(name=f"t{i}", **s) for i, s in enumerate(specs)]
    prm = dict(EPIE, iterations=2)
    t = default_shape(128, 3, 2)
    ref = make(ws, 2)
    assert kernels_of(lambda: api.rpie_batched(ref, tuning=t, **prm)) == FUSED
    runs, streams = [make(ws, 2), make(ws, 2)], [torch.cuda.Stream(), torch.cuda.Stream()]
    for run in runs:
        for j, w in zip(run, api.rpie_batched(make(ws, 2), tuning=t, **prm)):
            j["workspace"] = w
    torch.cuda.synchronize()
    errors = []

    def work(k):
        try:
            api.rpie_batched(runs[k], stream=streams[k], tuning=t, **prm)
        except Exception as e:  # surfaced below
            errors.append(e)
    th = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for x in th:
        x.start()
    for x in th:
        x.join()
    torch.cuda.synchronize()
    assert not errors
    for run in runs:
        for a, b in zip(run, ref):
            assert torch.equal(a["obj"], b["obj"]) and torch.equal(a["probe"], b["probe"])
            assert torch.equal(a["err"], b["err"])


@pytest.mark.parametrize("N,M,H,W", [(128, 1, 320, 320), (128, 8, 256, 384), (64, 3, 160, 160), (32, 5, 96, 96),
                                     (256, 3, 300, 290)])
def test_single_sweep_as_launches(N, M, H, W):
    w = wl.small_case(28, H, N, M, 6, W=W, name="one")
    prm = dict(EPIE, iterations=1)
    out = []
    assert kernels_of(lambda: out.append(alone(w, prm))) == FUSED
    o = run_oracle(w, prm)
    assert rel_l2(out[0]["O"], o["O"]) < 1e-4 and rel_l2(out[0]["P"], o["P"]) < 1e-4 and out[0]["status"] == 0


@pytest.mark.parametrize("jobs,M", [(9, 3), (12, 5), (15, 2), (40, 4), (75, 1)])
def test_batches_of_192_by_default(jobs, M):
    """... with ragged scans; 75 are more than two streams' lanes."""
    from paper_2205_04295_amd import api
    ws = [wl.small_case(700 + b % 4, 192 + 17, 192, M, 1 + b % 4, W=192 + 30, name=f"d{b % 4}") for b in range(jobs)]
    prm = dict(EPIE, iterations=2)
    got = make(ws, 2)
    k = kernels_of(lambda: api.rpie_batched(got, **prm))
    assert k == (SPLIT if jobs >= 16 else FUSED)
    check_against_alone(got[:4], ws[:4], prm)
    for b in range(4, jobs):
        assert rel_l2(got[b]["obj"].cpu().numpy(), got[b % 4]["obj"].cpu().numpy()) < 1e-6
    check_oracle(got[3], ws[3], prm)
