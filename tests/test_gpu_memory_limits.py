"""Contexts whose device memory has no room for the operand copies.

The copies of K, of right operands and of A in the layouts that the fast
products read are optional: where the caller's allocator refuses them, or a
bound region is too small for them, the products run from the matrices as they
are stored.  The results are those of the full context up to the order of
sums.
"""

import ctypes

import numpy as np
import pytest

from paper_1404_5776_amd import rtdm, synth
from tests._common import rel

pytestmark = pytest.mark.gpu

DT, STEPS = 0.05, 3


class CappedAllocator(rtdm.TorchAllocator):
    """The context's memory from torch, `cap` bytes of it at most."""

    def __init__(self, cap=None):
        super().__init__(0)
        self.cap, self.live, self.sizes, self.peak, self.log = cap, 0, {}, 0, []

    def _alloc(self, nbytes, user):
        if self.cap is not None and self.live + nbytes > self.cap:
            return None
        p = super()._alloc(nbytes, user)
        if p:
            self.sizes[p] = nbytes
            self.live += nbytes
            self.peak = max(self.peak, self.live)
            self.log.append(self.live)
        return p

    def _free(self, ptr, user):
        self.live -= self.sizes.pop(ptr)
        super()._free(ptr, user)


def _system(which):
    if which == "b13_etrs" or which == "b13":
        return synth.diamond_lattice((2, 2, 2), 13, 10.0, 12.0, seed=79, k0="local", h_model="mulliken")
    if which == "b4_runs":
        return synth.diamond_lattice((6, 6, 6), 4, 10.0, 12.0, seed=80, h_model="mulliken")
    return synth.config1()


def _options(which, s):
    return {"h_model": s.h_model, "propagator": "etrs" if which == "b13_etrs" else "em", "unit_check_every": 2}


def _load(which, cap=None):
    s = _system(which)
    print(f"[gpu] {which}: at most {cap} bytes", flush=True)
    ctx = rtdm.Context(0, memory="library", **_options(which, s))
    ctx.allocator = CappedAllocator(cap)
    rtdm.rtdm_set_allocator(ctx.h, ctx.allocator)
    rtdm.rtdm_set_geometry(ctx.h, s.xyz, s.nbf)
    rtdm.rtdm_set_ranges(ctx.h, s.R_HS, s.R_P, s.R_K)
    ctx.allocator.ranges_log = list(ctx.allocator.log)
    for name, m in (("S", s.S), ("H0", s.H0), ("K", s.K0)):
        rtdm.rtdm_upload_coo(ctx.h, name, m.rows, m.cols, m.data)
    ctx.b = s.b
    return s, ctx


def _run(s, ctx):
    rtdm.rtdm_build_inverse(ctx.h)
    rtdm.rtdm_apply_kick(ctx.h, (0.01, 0.0, 0.005))
    rtdm.rtdm_step(ctx.h, DT, STEPS)
    return _read(s, ctx)


def _read(s, ctx):
    W = rtdm.rtdm_download(ctx.h, "W", s.b)
    return (rtdm.rtdm_download(ctx.h, "K", s.b), rtdm.rtdm_download(ctx.h, "U", s.b), W,
            rtdm.rtdm_dipole_trace(ctx.h)[:, 4], rtdm.rtdm_observables(ctx.h)[3:4])


def _same(got, want):
    for g, w in zip(got, want):
        assert rel(g, w) <= 1e-12, rel(g, w)


# planes of the copies: K's right-operand form, the buffer of right operands, (ETRS) that of left ones
COPIES = {"b4_small": 2, "b4_runs": 4, "b13": 4, "b13_etrs": 6}
WHICH = list(COPIES)


@pytest.mark.parametrize("which", WHICH)
def test_an_allocator_without_room_for_the_copies(which):
    """Caps from one byte to two planes of K below the most that the full run
    held: the copies are refused when the ranges are set, or given back when a
    later call finds no room for its temporaries."""
    s, ctx = _load(which)
    setup = max(ctx.allocator.ranges_log[:-COPIES[which]])   # what every context holds before the copies, which come last
    want = _run(s, ctx)
    peak = ctx.allocator.peak
    nk = rtdm.rtdm_pattern(ctx.h, "K")[1].size * s.b * s.b * 8
    ctx.close()
    caps = [less for less in (1, nk // 2, nk, 3 * nk // 2, 2 * nk) if peak - less >= setup]
    assert caps
    for less in caps:
        s, ctx = _load(which, peak - less)
        got = _run(s, ctx)
        assert ctx.allocator.peak <= peak - less
        ctx.close()
        _same(got, want)


@pytest.mark.parametrize("which", WHICH)
def test_a_region_without_room_for_the_copies(which):
    """A region two planes of K smaller than the context's buffers, bound in
    the middle of a run: W of the last step, and the steps after it."""
    import torch
    s, ctx = _load(which)
    want1 = _run(s, ctx)
    rtdm.rtdm_step(ctx.h, DT, STEPS)
    want2 = _read(s, ctx)
    ctx.close()
    s, ctx = _load(which)
    rtdm.rtdm_reserve_trace(ctx.h, 64)
    rtdm.rtdm_build_inverse(ctx.h)
    rtdm.rtdm_apply_kick(ctx.h, (0.01, 0.0, 0.005))
    rtdm.rtdm_step(ctx.h, DT, STEPS)
    nk = rtdm.rtdm_pattern(ctx.h, "K")[1].size * s.b * s.b * 8
    live = rtdm.rtdm_workspace_size(ctx.h) - (64 << 20)
    region = torch.empty(live - nk, dtype=torch.uint8, device="cuda:0")
    rtdm.rtdm_bind_workspace(ctx.h, region.data_ptr(), region.numel())
    _same(_read(s, ctx), want1)
    rtdm.rtdm_step(ctx.h, DT, STEPS)
    _same(_read(s, ctx), want2)
    ctx.close()


@pytest.mark.parametrize("which", WHICH)
def test_a_region_that_the_trace_outgrows(which):
    """A region that holds the copies but not a trace grown by half of their
    size as well: the copies give way, the steps go on."""
    import torch
    s, ctx = _load(which)
    _run(s, ctx)
    rtdm.rtdm_step(ctx.h, DT, STEPS)
    want = _read(s, ctx)
    ctx.close()
    s, ctx = _load(which)
    rtdm.rtdm_build_inverse(ctx.h)
    rtdm.rtdm_apply_kick(ctx.h, (0.01, 0.0, 0.005))
    rtdm.rtdm_step(ctx.h, DT, STEPS)
    copies = COPIES[which] * rtdm.rtdm_pattern(ctx.h, "K")[1].size * s.b * s.b * 8
    live = rtdm.rtdm_workspace_size(ctx.h) - (64 << 20)
    grown = 64 << (copies // 2 // 64).bit_length() - 1     # a power of two: the largest trace below half of the copies
    region = torch.empty(live + grown // 2, dtype=torch.uint8, device="cuda:0")
    rtdm.rtdm_bind_workspace(ctx.h, region.data_ptr(), region.numel())
    rtdm.rtdm_reserve_trace(ctx.h, grown // 64)
    rtdm.rtdm_step(ctx.h, DT, STEPS)
    _same(_read(s, ctx), want)
    ctx.close()


@pytest.mark.parametrize("n", [65, 700])
def test_gradient_without_room_for_the_chunks_partial_sums(n):
    """The network's gradient is summed over chunks of samples whose partial
    sums are the last buffer it asks for; without them one chunk takes every
    sample: the same gradient up to the order of FP32 sums of n terms."""
    b = 4
    n_in, n_out = 4 + b * b, b * b
    rng = np.random.default_rng(85)
    desc, target = rng.normal(size=(n, n_in)).astype(np.float32), rng.normal(size=(n, n_out)).astype(np.float32)

    def run(cap):
        ctx = rtdm.Context(0, memory="library")
        ctx.allocator = CappedAllocator(cap)
        rtdm.rtdm_set_allocator(ctx.h, ctx.allocator)
        rtdm.rtdm_set_geometry(ctx.h, np.zeros((1, 3)), np.full(1, b, dtype=np.int32))
        rtdm.rtdm_mlp_init(ctx.h, 3)
        out = rtdm.rtdm_mlp_loss_grad(ctx.h, desc, target)
        live = ctx.allocator.live
        ctx.close()
        return out, live

    print(f"[gpu] gradient of {n} samples, capped", flush=True)
    (l0, g0), live = run(None)
    (l1, g1), less = run(live - 1)
    assert less < live
    assert l0 == l1
    assert np.abs(g1 - g0).max() <= n * np.finfo(np.float32).eps * np.abs(g0).max()
