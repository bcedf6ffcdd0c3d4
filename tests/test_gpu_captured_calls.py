"""Calls recorded into a caller's HIP graph and replayed between eager calls.

A context keeps K a second time in the layout that U K reads; whatever writes
K inside a graph has to write that copy too, at every replay, and a call that
was only recorded must not count as done.  Every sequence is compared with
the same calls issued eagerly, bit for bit.
"""

import numpy as np
import pytest

from paper_1404_5776_amd import rtdm, synth
from tests._common import gpu_context

pytestmark = pytest.mark.gpu

DT = 0.05


def _system(b):
    if b == 4:
        return synth.config1()
    return synth.diamond_lattice((2, 2, 2), 13, 10.0, 16.0, seed=71, k0="local", h_model="fixed")


def _blocks(ctx, b, seed):
    """Hermitian-pattern-free complex blocks of K's range on the GPU."""
    import torch
    n = rtdm.rtdm_pattern(ctx.h, "K")[1].size
    rng = np.random.default_rng(seed)
    v = 0.1 * (rng.uniform(-1, 1, size=(n, b, b)) + 1j * rng.uniform(-1, 1, size=(n, b, b)))
    return torch.from_numpy(v).cuda()


def _ready(s):
    """A context whose propagator is built (a fixed H keeps it) and a side stream."""
    import torch
    ctx = gpu_context(s, h_model="fixed")
    rtdm.rtdm_build_inverse(ctx.h)
    rtdm.rtdm_step(ctx.h, DT, 1)
    torch.cuda.synchronize()
    return ctx, torch.cuda.Stream()


def _record(stream, calls):
    import torch
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        calls()
    return g


def _eager(s, K, calls):
    ctx, st = _ready(s)
    rtdm.rtdm_upload(ctx.h, "K", K(ctx), st)
    calls(ctx, st)
    st.synchronize()
    out = rtdm.rtdm_download(ctx.h, "K", s.b)
    ctx.close()
    return out


@pytest.mark.parametrize("b", [4, 13])
def test_replayed_step_reads_the_k_of_an_upload_before_the_replay(b):
    s = _system(b)
    print(f"[gpu] captured step, b={b}", flush=True)
    want = _eager(s, lambda c: _blocks(c, b, 3), lambda c, st: rtdm.rtdm_step(c.h, DT, 2, st))
    ctx, st = _ready(s)
    rtdm.rtdm_upload(ctx.h, "K", _blocks(ctx, b, 2), st)
    rtdm.rtdm_step(ctx.h, DT, 1, st)
    g = _record(st, lambda: rtdm.rtdm_step(ctx.h, DT, 1, st))
    for _ in range(2):
        rtdm.rtdm_upload(ctx.h, "K", _blocks(ctx, b, 3), st)
        st.synchronize()
        for _ in range(2):
            g.replay()
        st.synchronize()
        import torch
        torch.cuda.synchronize()
        got = rtdm.rtdm_download(ctx.h, "K", b)
        assert np.array_equal(got, want), float(np.abs(got - want).max())
    ctx.close()


@pytest.mark.parametrize("b", [4, 13])
def test_step_after_a_replayed_product_into_k(b):
    """K = W U^dagger recorded, then steps, the replay, and a step that reads the K it wrote."""
    import torch
    s = _system(b)
    print(f"[gpu] captured product into K, b={b}", flush=True)

    def calls(c, st):
        rtdm.rtdm_step(c.h, DT, 1, st)
        rtdm.rtdm_upload(c.h, "W", _blocks(c, b, 5), st)
        rtdm.rtdm_multiply_noalloc(c.h, "K", "W", "U", 0, 1, 1.0, st)
        rtdm.rtdm_step(c.h, DT, 1, st)

    want = _eager(s, lambda c: _blocks(c, b, 3), calls)
    ctx, st = _ready(s)
    rtdm.rtdm_upload(ctx.h, "W", _blocks(ctx, b, 5), st)
    g = _record(st, lambda: rtdm.rtdm_multiply_noalloc(ctx.h, "K", "W", "U", 0, 1, 1.0, st))
    for _ in range(2):
        rtdm.rtdm_upload(ctx.h, "K", _blocks(ctx, b, 3), st)
        rtdm.rtdm_step(ctx.h, DT, 1, st)
        rtdm.rtdm_upload(ctx.h, "W", _blocks(ctx, b, 5), st)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        rtdm.rtdm_step(ctx.h, DT, 1, st)
        st.synchronize()
        got = rtdm.rtdm_download(ctx.h, "K", b)
        assert np.array_equal(got, want), float(np.abs(got - want).max())
    ctx.close()


@pytest.mark.parametrize("b", [4, 13])
def test_step_after_a_replayed_upload_of_k(b):
    import torch
    s = _system(b)
    print(f"[gpu] captured upload of K, b={b}", flush=True)
    want = _eager(s, lambda c: _blocks(c, b, 3), lambda c, st: rtdm.rtdm_step(c.h, DT, 1, st))
    ctx, st = _ready(s)
    K = _blocks(ctx, b, 2)
    torch.cuda.synchronize()
    g = _record(st, lambda: rtdm.rtdm_upload(ctx.h, "K", K, st))
    for _ in range(2):
        rtdm.rtdm_step(ctx.h, DT, 1, st)
        st.synchronize()
        K.copy_(_blocks(ctx, b, 3))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        rtdm.rtdm_step(ctx.h, DT, 1, st)
        st.synchronize()
        got = rtdm.rtdm_download(ctx.h, "K", b)
        assert np.array_equal(got, want), float(np.abs(got - want).max())
    ctx.close()


@pytest.mark.parametrize("b", [4, 13])
def test_a_kick_that_was_only_recorded_has_not_been_applied(b):
    s = _system(b)
    print(f"[gpu] recorded kick, b={b}", flush=True)
    want = _eager(s, lambda c: _blocks(c, b, 3), lambda c, st: rtdm.rtdm_step(c.h, DT, 1, st))
    ctx, st = _ready(s)
    rtdm.rtdm_upload(ctx.h, "K", _blocks(ctx, b, 3), st)
    st.synchronize()
    g = _record(st, lambda: rtdm.rtdm_apply_kick(ctx.h, (0.02, 0.0, 0.01), st))
    rtdm.rtdm_step(ctx.h, DT, 1, st)
    st.synchronize()
    got = rtdm.rtdm_download(ctx.h, "K", b)
    assert np.array_equal(got, want), float(np.abs(got - want).max())
    del g
    ctx.close()


# (recorded product, product issued eagerly on another stream meanwhile): they share no slot that either writes
PRODUCTS = [(("A", "X", "H0", 0, 0, 1.0), ("W", "U", "K", 0, 0, 1.0)),
            (("W", "U", "K", 0, 0, 1.0), ("A", "X", "H0", 0, 0, 1.0)),
            (("K", "W", "U", 0, 1, 1.0), ("A", "X", "H0", 0, 0, 1.0)),
            (("U", "A", "X", 0, 0, 0.5j), ("W", "X", "K", 0, 0, 1.0)),
            (("W", "X", "K", 0, 0, 0.5j), ("U", "A", "X", 0, 0, 1.0))]


@pytest.mark.parametrize("which", ["b4", "b13", "b13_etrs"])
@pytest.mark.parametrize("job,other", PRODUCTS)
def test_a_replayed_product_shares_no_buffer_with_eager_ones(which, job, other):
    """Replays of a recorded product overlap eager products on another stream:
    every result is bit for bit that of the call by itself.  Recorded products
    read their operands by rows instead of laying them out in a buffer of the
    context's (b = 4: row runs that fill the chip; b = 13: pair layout)."""
    import torch
    s = (synth.diamond_lattice((6, 6, 6), 4, 10.0, 12.0, seed=83, h_model="fixed") if which == "b4" else
         synth.diamond_lattice((2, 2, 2), 13, 10.0, 16.0, seed=84, k0="local", h_model="fixed"))
    ctx = gpu_context(s, h_model="fixed", propagator="etrs" if which == "b13_etrs" else "em")
    rtdm.rtdm_build_inverse(ctx.h)
    rtdm.rtdm_step(ctx.h, DT, 1)
    W = rtdm.rtdm_download(ctx.h, "W", s.b)
    rtdm.rtdm_upload(ctx.h, "W", W)
    want = []
    for j in (job, other):
        rtdm.rtdm_multiply(ctx.h, *j)
        want.append(rtdm.rtdm_download(ctx.h, j[0], s.b))
    a, c = torch.cuda.Stream(), torch.cuda.Stream()
    g = _record(a, lambda: rtdm.rtdm_multiply_noalloc(ctx.h, *job, a))
    for rep in range(4):
        print(f"[gpu] {which} recorded {job[0]} = {job[1]} {job[2]} rep={rep}", flush=True)
        for j in (job, other):
            rtdm.rtdm_upload(ctx.h, j[0], np.zeros_like(want[0] if j is job else want[1]))
        torch.cuda.synchronize()
        for _ in range(4):
            with torch.cuda.stream(a):
                g.replay()
            rtdm.rtdm_multiply(ctx.h, *other, c)
        torch.cuda.synchronize()
        for j, w in zip((job, other), want):
            assert np.array_equal(rtdm.rtdm_download(ctx.h, j[0], s.b), w), (j, rep)
    ctx.close()
