"""Calls of one context on several streams: asynchronous, and in order where
they share the buffers that products lay their operands out in.

A stream is held by a kernel that waits on the GPU (torch.cuda._sleep); what
the host may return from, and what has to be complete when a later call is,
is then read from the streams.
"""

import numpy as np
import pytest

from paper_1404_5776_amd import rtdm, synth
from tests._common import gpu_context

pytestmark = pytest.mark.gpu

HOLD = 400_000_000      # GPU clocks: some tenths of a second


def _b13(use_graph=0):
    s = synth.diamond_lattice((2, 2, 2), 13, 10.0, 16.0, seed=73, k0="local", h_model="fixed")
    ctx = gpu_context(s, h_model="fixed", use_graph=use_graph)
    rtdm.rtdm_build_inverse(ctx.h)
    rtdm.rtdm_step(ctx.h, 0.05, 1)
    return s, ctx


def test_a_product_behind_a_step_on_another_stream_does_not_block_the_host():
    import torch
    s, ctx = _b13()
    rtdm.rtdm_multiply(ctx.h, "A", "X", "H0")
    want = rtdm.rtdm_download(ctx.h, "A", s.b)
    a, c = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    print("[gpu] step on one stream, product on another", flush=True)
    with torch.cuda.stream(a):
        torch.cuda._sleep(HOLD)
    rtdm.rtdm_step(ctx.h, 0.05, 1, a)
    rtdm.rtdm_multiply_noalloc(ctx.h, "A", "X", "H0", 0, 0, 1.0, c)
    held = not a.query()
    torch.cuda.synchronize()
    assert held, "the call waited for the other stream on the host"
    assert np.array_equal(rtdm.rtdm_download(ctx.h, "A", s.b), want)
    ctx.close()


def test_steps_on_alternating_streams_do_not_block_the_host():
    import torch
    s, ctx = _b13()
    K0 = rtdm.rtdm_download(ctx.h, "K", s.b)
    rtdm.rtdm_step(ctx.h, 0.05, 4)
    want = rtdm.rtdm_download(ctx.h, "K", s.b)
    rtdm.rtdm_upload(ctx.h, "K", K0)
    a, c = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    print("[gpu] steps on two streams ordered by the caller's events", flush=True)
    with torch.cuda.stream(a):
        torch.cuda._sleep(HOLD)
    hold = torch.cuda.Event()
    hold.record(a)
    for k in range(4):
        x, y = (a, c) if k % 2 == 0 else (c, a)
        rtdm.rtdm_step(ctx.h, 0.05, 1, x)
        e = torch.cuda.Event()
        e.record(x)
        y.wait_event(e)
    held = not hold.query()
    torch.cuda.synchronize()
    assert held, "a step waited for the other stream on the host"
    assert np.array_equal(rtdm.rtdm_download(ctx.h, "K", s.b), want)
    ctx.close()


def test_a_product_behind_graph_steps_on_the_null_stream_does_not_block_the_host():
    import torch
    s, ctx = _b13(use_graph=1)
    h = torch.cuda.Stream()
    rtdm.rtdm_step(ctx.h, 0.05, 2, 0)                 # captured and replayed on the library's own stream
    rtdm.rtdm_multiply_noalloc(ctx.h, "A", "X", "H0", 0, 0, 1.0, h)
    torch.cuda.synchronize()
    print("[gpu] graph steps on the null stream, product on another", flush=True)
    want = rtdm.rtdm_download(ctx.h, "A", s.b)
    torch.cuda.synchronize()
    torch.cuda._sleep(HOLD)                            # torch's default stream is the null stream
    e = torch.cuda.Event()
    e.record()
    rtdm.rtdm_step(ctx.h, 0.05, 2, 0)
    rtdm.rtdm_multiply_noalloc(ctx.h, "A", "X", "H0", 0, 0, 1.0, h)
    held = not e.query()
    torch.cuda.synchronize()
    assert held, "the call waited for the device on the host"
    assert np.array_equal(rtdm.rtdm_download(ctx.h, "A", s.b), want)
    ctx.close()


def _order(first, second, streams):
    """`first` behind a held stream, `second` at once on another: whether the first is complete when the second is."""
    import torch
    a, c = streams
    torch.cuda.synchronize()
    with torch.cuda.stream(a):
        torch.cuda._sleep(HOLD)
    first(a)
    done = torch.cuda.Event()
    done.record(a)
    second(c)
    held = not done.query()
    end = torch.cuda.Event()
    end.record(c)
    end.synchronize()
    return held, done.query()


def _b4():
    s = synth.diamond_lattice((6, 6, 6), 4, 10.0, 12.0, seed=74, h_model="fixed")
    ctx = gpu_context(s, h_model="fixed")
    rtdm.rtdm_build_inverse(ctx.h)
    rtdm.rtdm_step(ctx.h, 0.05, 1)
    return s, ctx


def test_products_of_an_etrs_context_on_two_streams_run_in_turn():
    """b = 13, ETRS: A T and U K with an imaginary factor lay both operands out
    in the context's buffers and return at once."""
    import torch
    s = synth.diamond_lattice((2, 2, 2), 13, 10.0, 16.0, seed=76, k0="local", h_model="fixed")
    ctx = gpu_context(s, h_model="fixed", propagator="etrs")
    rtdm.rtdm_build_inverse(ctx.h)
    rtdm.rtdm_step(ctx.h, 0.05, 1)
    jobs = [("U", "A", "X", 1j), ("W", "X", "K", 0.5j)]
    ref = []
    for c, a, b, al in jobs:
        rtdm.rtdm_multiply(ctx.h, c, a, b, 0, 0, al)
        ref.append(rtdm.rtdm_download(ctx.h, c, s.b))
    streams = [torch.cuda.Stream() for _ in jobs]
    call = [lambda st, j=j: rtdm.rtdm_multiply(ctx.h, j[0], j[1], j[2], 0, 0, j[3], st) for j in jobs]
    for k in (0, 1):
        print(f"[gpu] ETRS products on two streams, {jobs[k][0]} first", flush=True)
        held, done = _order(call[k], call[1 - k], streams)
        assert held and done, (held, done)
        torch.cuda.synchronize()
        for (c, *_), r in zip(jobs, ref):
            assert np.array_equal(rtdm.rtdm_download(ctx.h, c, s.b), r)
    for rep in range(8):
        print(f"[gpu] ETRS products on two streams rep={rep}", flush=True)
        for _ in range(4):
            for f, st in zip(call, streams):
                f(st)
        torch.cuda.synchronize()
        for (c, *_), r in zip(jobs, ref):
            assert np.array_equal(rtdm.rtdm_download(ctx.h, c, s.b), r), (c, rep)
    ctx.close()


def test_a_recorded_product_leaves_the_turn_of_those_in_flight():
    """A product in flight on one stream, another recorded into a graph on a
    second one, then an eager product on that second stream: it waits for the
    first, as if nothing had been recorded."""
    import torch
    s, ctx = _b4()
    a, c = torch.cuda.Stream(), torch.cuda.Stream()
    rtdm.rtdm_multiply(ctx.h, "A", "X", "H0")
    want = rtdm.rtdm_download(ctx.h, "A", s.b)
    rtdm.rtdm_multiply(ctx.h, "W", "U", "K")
    W = rtdm.rtdm_download(ctx.h, "W", s.b)
    graphs = []

    def second(st):
        g = torch.cuda.CUDAGraph()
        with torch.cuda.stream(st):
            g.capture_begin()
            rtdm.rtdm_multiply_noalloc(ctx.h, "A", "X", "H0", 0, 0, 1.0, st)
            g.capture_end()
        graphs.append(g)
        rtdm.rtdm_multiply(ctx.h, "A", "X", "H0", 0, 0, 1.0, st)

    print("[gpu] a product recorded between two eager ones", flush=True)
    held, done = _order(lambda st: rtdm.rtdm_multiply(ctx.h, "W", "U", "K", 0, 0, 1.0, st), second, (a, c))
    assert held and done, (held, done)
    torch.cuda.synchronize()
    assert np.array_equal(rtdm.rtdm_download(ctx.h, "A", s.b), want)
    assert np.array_equal(rtdm.rtdm_download(ctx.h, "W", s.b), W)
    del graphs
    ctx.close()


@pytest.mark.parametrize("call", ["observables", "unitarity", "inverse_error"])
def test_a_measurement_behind_a_product_on_another_stream_waits_its_turn(call):
    """The products of the measures lay their right operand out where the one
    in flight does; the calls return host values, so the other is complete."""
    import torch
    s, ctx = _b4()
    measure = getattr(rtdm, "rtdm_" + call)
    want = measure(ctx.h)
    rtdm.rtdm_multiply(ctx.h, "A", "X", "H0")
    A = rtdm.rtdm_download(ctx.h, "A", s.b)
    streams = [torch.cuda.Stream() for _ in range(2)]
    print(f"[gpu] {call} behind a product on another stream", flush=True)
    torch.cuda.synchronize()
    with torch.cuda.stream(streams[0]):
        torch.cuda._sleep(HOLD)
    rtdm.rtdm_multiply(ctx.h, "A", "X", "H0", 0, 0, 1.0, streams[0])
    done = torch.cuda.Event()
    done.record(streams[0])
    assert not done.query()
    got = measure(ctx.h, streams[1])
    assert done.query()
    assert np.array_equal(got, want)
    assert np.array_equal(rtdm.rtdm_download(ctx.h, "A", s.b), A)
    ctx.close()


@pytest.mark.parametrize("use_graph", [0, 1])
@pytest.mark.parametrize("capturing", [False, True])
def test_a_product_behind_steps_on_the_null_stream_waits_its_turn(use_graph, capturing):
    """A step held on the null stream (replayed: on the library's own), then a
    product at once on a stream that is not in order with it, also while a third
    stream is captured; and a step on the null stream behind that product."""
    import torch
    s, ctx = _b13(use_graph)
    K0 = rtdm.rtdm_download(ctx.h, "K", s.b)
    rtdm.rtdm_multiply(ctx.h, "A", "X", "H0")
    A = rtdm.rtdm_download(ctx.h, "A", s.b)
    rtdm.rtdm_step(ctx.h, 0.05, 2, 0)
    K = rtdm.rtdm_download(ctx.h, "K", s.b)
    rtdm.rtdm_upload(ctx.h, "K", K0)
    c, other = torch.cuda.Stream(), torch.cuda.Stream()
    x = torch.zeros(8, device="cuda:0")
    torch.cuda.synchronize()
    print(f"[gpu] steps on the null stream, product on another, graph={use_graph} capturing={capturing}", flush=True)
    torch.cuda._sleep(HOLD)                            # torch's default stream is the null stream
    rtdm.rtdm_step(ctx.h, 0.05, 1, 0)
    done = torch.cuda.Event()
    done.record()
    if capturing:
        g = torch.cuda.CUDAGraph()
        with torch.cuda.stream(other):
            g.capture_begin()
            x += 1
    rtdm.rtdm_multiply_noalloc(ctx.h, "A", "X", "H0", 0, 0, 1.0, c)
    if capturing:
        with torch.cuda.stream(other):
            g.capture_end()
    held = not done.query()
    end = torch.cuda.Event()
    end.record(c)
    end.synchronize()
    assert held and done.query(), "the product did not run behind the step"
    with torch.cuda.stream(c):
        torch.cuda._sleep(HOLD)
    rtdm.rtdm_multiply_noalloc(ctx.h, "A", "X", "H0", 0, 0, 1.0, c)
    done.record(c)
    rtdm.rtdm_step(ctx.h, 0.05, 1, 0)
    held = not done.query()
    end.record()
    end.synchronize()
    assert held and done.query(), "the step did not run behind the product"
    torch.cuda.synchronize()
    assert np.array_equal(rtdm.rtdm_download(ctx.h, "A", s.b), A)
    assert np.array_equal(rtdm.rtdm_download(ctx.h, "K", s.b), K)
    if capturing:
        g.replay()
        torch.cuda.synchronize()
        assert float(x.sum()) == 8.0
    ctx.close()
