"""Kick sets in every precision of the products: the trace of each set,
Hermiticity error included, equals a one-kick run's.

The Hermiticity sums of a step are finished after the last kick's products, so
nothing that a product uses on the way may lie over them.
"""

import numpy as np
import pytest

from paper_1404_5776_amd import rtdm
from tests._common import small_clusters

pytestmark = pytest.mark.gpu

KICKS = [(0.01, 0.0, 0.0), (0.0, 0.02, 0.0), (0.0, 0.0, 0.03)]
DT, STEPS = 0.05, 3


@pytest.mark.parametrize("b", [4, 13])
@pytest.mark.parametrize("precision", ["fp64", "fp32", "bf16x3", "fp16x2"])
def test_every_sets_hermiticity_error_is_that_of_a_one_kick_run(precision, b):
    systems = small_clusters(b)[:2]
    print(f"[gpu] kick sets, {precision}, b={b}", flush=True)
    ctx = rtdm.Context(0, h_model="fixed", precision=precision, n_kicks=len(KICKS))
    ctx.load_kick_sets(systems, KICKS)
    rtdm.rtdm_build_inverse(ctx.h)
    rtdm.rtdm_apply_kicks(ctx.h, ctx.kick_vectors)
    rtdm.rtdm_step(ctx.h, DT, STEPS)
    got = []
    for k in range(len(KICKS)):
        rtdm.rtdm_select_kick(ctx.h, k)
        got.append((rtdm.rtdm_dipole_trace(ctx.h), rtdm.rtdm_observables(ctx.h)))
    ctx.close()
    for k, kap in enumerate(KICKS):
        one = rtdm.Context(0, h_model="fixed", precision=precision)
        one.load_batch(systems, [[(0.0, 0.0, 0.0)]] * len(systems))
        rtdm.rtdm_build_inverse(one.h)
        rtdm.rtdm_apply_kick(one.h, kap)
        rtdm.rtdm_step(one.h, DT, STEPS)
        tr, ob = rtdm.rtdm_dipole_trace(one.h), rtdm.rtdm_observables(one.h)
        one.close()
        assert np.all(tr[:, 5] > 0.0), (k, tr[:, 5])
        assert np.array_equal(got[k][0][:, :6], tr[:, :6]), (k, got[k][0][:, 5], tr[:, 5])
        assert np.array_equal(got[k][1][:5], ob[:5]), k
