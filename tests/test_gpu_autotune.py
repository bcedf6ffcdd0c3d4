"""The launch-shape tuner: what it chooses from."""

import numpy as np
import pytest

from paper_1404_5776_amd import rtdm, synth
from tests._common import gpu_context

pytestmark = pytest.mark.gpu


def test_candidates_are_those_that_differ():
    """343 atoms on the row-run kernels: these have one workgroup shape, so the
    waves per workgroup stay (a choice between equals would be one by noise);
    the default tile of 512 rows is a candidate, and 1,024 rows are the same
    order (all rows)."""
    xyz = synth.cluster_positions(343, np.random.default_rng(75))
    s = synth.build_system("c343", xyz, 13, 6.0, 9.0, 75, k0="local")
    seen = []
    for rep in range(6):
        ctx = gpu_context(s)
        rtdm.rtdm_build_inverse(ctx.h)
        rtdm.rtdm_step(ctx.h, s.dt, 1)
        seen.append(rtdm.rtdm_autotune(ctx.h))
        ctx.close()
    print(f"[gpu] autotune of 343 atoms: {seen}", flush=True)
    assert all(w == 16 and t in (64, 256, 512) for w, t in seen), seen


def test_one_order_leaves_nothing_to_choose():
    """40 atoms: every tile is the same order.  The smallest is reported each
    time, K and W stay what the step left."""
    xyz = synth.cluster_positions(40, np.random.default_rng(76))
    s = synth.build_system("c40", xyz, 13, 6.0, 9.0, 76, k0="exact")
    ctx = gpu_context(s)
    rtdm.rtdm_build_inverse(ctx.h)
    rtdm.rtdm_step(ctx.h, s.dt, 1)
    K, W = (rtdm.rtdm_download(ctx.h, m, s.b) for m in "KW")
    assert [rtdm.rtdm_autotune(ctx.h) for _ in range(6)] == [(16, 64)] * 6
    assert np.array_equal(rtdm.rtdm_download(ctx.h, "K", s.b), K)
    assert np.array_equal(rtdm.rtdm_download(ctx.h, "W", s.b), W)
    ctx.close()
