"""The slot W after steps: a step leaves U K in the form its second product reads
(b = 13), and what reads the slot has to see it by rows.
"""

import numpy as np
import pytest

from paper_1404_5776_amd import rtdm, synth
from tests._common import gpu_context

pytestmark = pytest.mark.gpu

DT = 0.05


def _context(b, **opts):
    s = synth.diamond_lattice((2, 2, 2), b, 10.0, 12.0, seed=87, k0="local", h_model="fixed")
    ctx = gpu_context(s, h_model="fixed", **opts)
    rtdm.rtdm_build_inverse(ctx.h)
    rtdm.rtdm_apply_kick(ctx.h, (0.01, 0.0, 0.005))
    return ctx


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("b", [4, 13])
def test_a_product_reads_w_of_the_last_step(b, precision):
    """W U^dagger of the slots right after steps, against the same with W
    downloaded in between."""
    got = []
    for through_host in (True, False):
        ctx = _context(b, precision=precision)
        rtdm.rtdm_step(ctx.h, DT, 2)
        if through_host:
            rtdm.rtdm_download(ctx.h, "W", b)
        rtdm.rtdm_multiply(ctx.h, "K", "W", "U", 0, 1)
        got.append(rtdm.rtdm_download(ctx.h, "K", b))
        ctx.close()
    assert np.array_equal(got[0], got[1])


@pytest.mark.parametrize("b", [4, 13])
def test_w_downloaded_between_replayed_steps(b):
    """Graph steps, W, graph steps, W: each the W of the last step, as after eager steps."""
    got = []
    for use_graph in (0, 1):
        ctx = _context(b, use_graph=use_graph)
        ws = []
        for _ in range(3):
            rtdm.rtdm_step(ctx.h, DT, 3)
            ws.append(rtdm.rtdm_download(ctx.h, "W", b))
        got.append(ws)
        ctx.close()
    for eager, replayed in zip(*got):
        assert np.array_equal(eager, replayed)
    assert not np.array_equal(got[0][0], got[0][1])
