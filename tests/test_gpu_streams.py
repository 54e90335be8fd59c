"""The library's weight and forward streams go with the caller's stream: nets on
one share them, nets on two do not wait for each other; nets issued from two
threads on streams of their own, and a graph captured beside them, give what
they give alone."""
import threading

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

T = 6


def make(P, batch, seed):
    from paper_1912_12675_amd import synth
    wl = synth.resnet20_workload(batch=batch, seed=seed)
    net = P.Net(wl.ops, batch, wl.in_shape, wl.stage_end, [4, 3, 2, 1])
    net.load_params(synth.init_params(wl))
    xs, ys = synth.batches(wl, T, batch)
    return net, wl, torch.from_numpy(xs).cuda(), torch.from_numpy(ys).cuda()


def run(P, made, stream, steps_only=False):
    net, wl, xs, ys = made
    st = np.tile(np.array([3, 2, 1, 0], dtype=np.int32), (T, 1))
    losses = torch.zeros(T, device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        if steps_only:
            for t in range(T):
                net.step(t, st[t], wl.lr, xs[t], ys[t])
        else:
            net.pipeline_run(0, st, wl.lr, xs, ys, losses)
    stream.synchronize()
    return net.params(T)


def test_two_threads():
    from paper_1912_12675_amd import psw as P
    print("streams: two threads", flush=True)
    alone = [run(P, make(P, b, s), torch.cuda.Stream()) for b, s in ((8, 1), (12, 2))]
    made = [make(P, 8, 1), make(P, 12, 2)]
    got, errors = [None, None], []

    def work(i):
        try:
            got[i] = run(P, made[i], torch.cuda.Stream(), steps_only=i == 1)
        except Exception as e:  # reported below: a thread's exception does not fail a test
            errors.append(e)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for a, b in zip(alone, got):
        assert torch.equal(a, b)


def test_two_callers_do_not_wait_for_each_other():
    """With one net's stream held (by a kernel that spins for a bounded time), a net on another stream finishes
    its steps.  A process has four hardware queues, and two streams that share one do wait: some of the stream
    pairs tried have queues apart, and one is enough."""
    from paper_1912_12675_amd import psw as P
    print("streams: two callers", flush=True)
    start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda._sleep(1000)
    start.record()
    torch.cuda._sleep(1_000_000)
    end.record()
    torch.cuda.synchronize()
    cycles = int(250.0 / max(start.elapsed_time(end), 1e-3) * 1_000_000)  # a quarter of a second

    def step(m, t, stream):
        net, wl, xs, ys = m
        with torch.cuda.stream(stream):
            net.step(t, [3, 2, 1, 0], wl.lr, xs[t], ys[t])

    held, free = make(P, 8, 1), make(P, 8, 2)
    torch.cuda.synchronize()
    apart = False
    for t in range(T):
        a, b = torch.cuda.Stream(), torch.cuda.Stream()
        with torch.cuda.stream(a):
            torch.cuda._sleep(cycles)
            awake = a.record_event()
        step(held, t, a)
        step(free, t, b)
        b.synchronize()
        apart = apart or not awake.query()
        torch.cuda.synchronize()
    assert apart


def test_more_callers_than_pairs():
    """Steps of one net on more streams than the library keeps pairs for: pairs are handed on."""
    from paper_1912_12675_amd import psw as P
    print("streams: many callers", flush=True)
    ref = run(P, make(P, 8, 1), torch.cuda.Stream(), steps_only=True)
    net, wl, xs, ys = make(P, 8, 1)
    other = make(P, 12, 2)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(11)]
    for s in streams[:5]:  # pairs of other callers, one with work pending
        run(P, make(P, 12, 2), s, steps_only=True)
    with torch.cuda.stream(streams[5]):
        other[0].step(0, [3, 2, 1, 0], other[1].lr, other[2][0], other[3][0])
    for t in range(T):
        s = streams[5 + t]
        with torch.cuda.stream(s):
            net.step(t, [3, 2, 1, 0], wl.lr, xs[t], ys[t])
        s.synchronize()
    assert torch.equal(net.params(T), ref)


def test_streams_outlive_one_net():
    from paper_1912_12675_amd import psw as P
    print("streams: a net destroyed beside another", flush=True)
    ref = run(P, make(P, 8, 1), torch.cuda.Stream())
    first, second = make(P, 12, 2), make(P, 8, 1)
    run(P, first, torch.cuda.Stream())
    del first
    assert torch.equal(run(P, second, torch.cuda.Stream()), ref)
    del second
    assert torch.equal(run(P, make(P, 8, 1), torch.cuda.Stream()), ref)  # the streams are made again


@pytest.mark.parametrize("pipeline", [False, True])
def test_caller_captures_beside_another_net(pipeline):
    """A step captured into the caller's graph, with another net's step issued in
    another thread before the capture ends: neither takes the other's work in."""
    from paper_1912_12675_amd import psw as P
    print("streams: the caller's capture", flush=True)
    eager, other = make(P, 8, 1), make(P, 12, 2)
    zero = np.zeros((T, 4), dtype=np.int32)
    losses = torch.zeros(T, device="cuda")

    def step(m):
        net, wl, xs, ys = m
        if pipeline:
            net.pipeline_run(0, zero[:1], wl.lr, xs[:1], ys[:1], losses)
        else:
            net.step(0, zero[0], wl.lr, xs[0], ys[0])

    step(eager)
    torch.cuda.synchronize()
    ref = eager[0].params(1)
    ref_other = run(P, make(P, 12, 2), torch.cuda.Stream(), steps_only=True)

    made = make(P, 8, 1)
    net = made[0]
    start = net.ring.clone()
    net._ensure_pipeline_set()  # bound before the capture
    errors, theirs = [], torch.cuda.Stream()

    def beside():
        try:
            onet, owl, xs, ys = other
            with torch.cuda.stream(theirs):
                for t in range(T):
                    onet.step(t, [3, 2, 1, 0], owl.lr, xs[t], ys[t])
            theirs.synchronize()
        except Exception as e:  # reported below
            errors.append(e)

    thread = threading.Thread(target=beside)
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g, capture_error_mode="thread_local"):
        step(made)
        thread.start()
        thread.join()
    assert not errors, errors
    torch.cuda.synchronize()
    assert torch.equal(other[0].params(T), ref_other)
    for _ in range(3):
        net.ring.copy_(start)
        net.momentum.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(net.params(1), ref)
        step_again = make(P, 8, 1)
        step(step_again)  # eager work between the replays
        torch.cuda.synchronize()
        assert torch.equal(step_again[0].params(1), ref)
