"""Persistent sweeps on several streams: calls of fewer jobs than XCDs run side
by side and give the bits of calls made alone, a long call lets other streams'
kernels in between its launches, captured calls may be replayed side by side."""
import time

import pytest
import torch

from synth import workloads as wl

from gpu_util import need_gpu, to_dev

pytestmark = pytest.mark.gpu

EPIE = dict(alpha_obj=0.9, alpha_probe=0.9, beta=1.0, gamma=1.0)


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


def job(N, M, J, seed=0):
    d = to_dev(wl.small_case(1000 + seed, N + 40, N, M, J, W=N + 52, name=f"c{seed}"))
    return dict(obj=d["obj"], probe=d["probe"], pos=d["pos"], intens=d["I"])


def copy(j):
    return dict(j, obj=j["obj"].clone(), probe=j["probe"].clone())


def same(a, b):
    return torch.equal(a["obj"], b["obj"]) and torch.equal(a["probe"], b["probe"])


def run(j, stream, T):
    from paper_2205_04295_amd import api
    j["workspace"] = api.rpie(j["obj"], j["probe"], j["pos"], j["intens"], workspace=j.get("workspace"),
                              stream=stream, iterations=T, **EPIE)


@pytest.mark.parametrize("N,M,J,T", [(64, 1, 50, 10), (256, 3, 40, 5)])
def test_two_streams_run_side_by_side(N, M, J, T):
    """Two calls on two streams take about as long as one (measured 1.02 times;
    one after the other would be 2).  Streams may share one of the runtime's
    hardware queues, which takes their kernels one after the other: of three
    pairs the best counts."""
    js = [job(N, M, J, s) for s in range(2)]
    streams = [torch.cuda.Stream() for _ in range(4)]
    ref = [copy(j) for j in js]
    for r in ref:
        run(r, torch.cuda.current_stream(), T)
    torch.cuda.synchronize()

    for j in js:
        j["workspace"] = torch.empty_like(ref[0]["workspace"])

    def took(k):
        best = 1e9
        for rep in range(9):
            out = [copy(j) for j in js[:k]]
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for o, s in zip(out, (streams[0], streams[1 + rep % 3])):
                run(o, s, T)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t0)
            assert all(same(o, r) for o, r in zip(out, ref))
        return best
    one, two = took(1), took(2)
    print(f"{N}^2 x {M}: one {one * 1e3:.2f} ms, two {two * 1e3:.2f} ms")
    assert two < 1.5 * one


def test_long_call_lets_other_kernels_in():
    """... on a stream of another hardware queue: one of three at least."""
    j = job(256, 3, 100)
    x = torch.ones(1 << 24, device="cuda")
    s = torch.cuda.Stream()
    run(j, s, 1)
    others = [torch.cuda.Stream() for _ in range(3)]
    for other in others:
        with torch.cuda.stream(other):
            x.mul_(2.0)
        other.synchronize()
    before = []
    for other in others:
        torch.cuda.synchronize()
        run(j, s, 60)               # 6000 positions, some 85 ms
        with torch.cuda.stream(other):
            x.mul_(0.5)             # workgroups for every XCD
        other.synchronize()
        before.append(not s.query())  # ... were done before the call was
    torch.cuda.synchronize()
    print(before)
    assert any(before) and float(x[123]) == 1.0


def test_batches_of_several_sizes_on_four_streams():
    """1 to 8 jobs a call, so calls share XCDs or not; every job ends as in a
    call of its own batch alone."""
    from paper_2205_04295_amd import api
    sets = [[job(64, 2, 12, 1)], [job(128, 2, 8, 2), job(32, 3, 20, 3)], [job(64, 1, 9, k) for k in range(3)],
            [job(256, 2, 3, 4), job(64, 1, 30, 5), job(128, 1, 5, 6), job(64, 4, 7, 7)] * 2]
    ref = [[copy(j) for j in s] for s in sets]
    for r in ref:
        api.rpie_batched(r, iterations=2, **EPIE)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in sets]
    for rep in range(3):
        got = [[copy(j) for j in s] for s in sets]
        torch.cuda.synchronize()
        keep = [api.rpie_batched(g, stream=streams[(k + rep) % 4], iterations=2, **EPIE) for k, g in enumerate(got)]
        torch.cuda.synchronize()
        del keep
        for g, r in zip(got, ref):
            for a, b in zip(g, r):
                assert same(a, b)


def test_graphs_replayed_side_by_side():
    from paper_2205_04295_amd import api, graph
    sets = [[job(128, 2, 6, 10 + k) for k in range(n)] for n in (1, 2, 12)]
    got = [[copy(j) for j in s] for s in sets]
    ref = [[copy(j) for j in s] for s in sets]
    graphs = [graph.capture_batched(g, iterations=1, **EPIE) for g in got]
    streams = [torch.cuda.Stream() for _ in sets]
    for rep in range(3):
        torch.cuda.synchronize()
        for g, s in zip(graphs, streams):
            with torch.cuda.stream(s):
                g.replay()
        torch.cuda.synchronize()
        for r in ref:
            api.rpie_batched(r, iterations=1, **EPIE)
        torch.cuda.synchronize()
        for g, r in zip(got, ref):
            for a, b in zip(g, r):
                assert same(a, b), rep
