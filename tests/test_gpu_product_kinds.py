"""Which product kinds the allocation-free call takes after rtdm_set_ranges."""

import numpy as np
import pytest

from oracle import oracle as O
from paper_1404_5776_amd import rtdm, synth
from tests._common import TOL, rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b,n", [(4, 40), (4, 4200), (13, 40)])
def test_the_unitarity_product_is_scheduled_where_steps_check_it(b, n):
    """U^dagger V (a real operand in U's place) without a rtdm_multiply before
    it, at b = 4 also where the check itself runs over row runs."""
    rng = np.random.default_rng(3)
    g = synth.CLUSTER_DENSITY ** (-1.0 / 3.0)
    m = int(np.ceil(n ** (1.0 / 3.0)))
    p = np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing="ij"), -1).reshape(-1, 3)[:n] * g
    xyz = np.ascontiguousarray(p + rng.uniform(-0.4, 0.4, size=p.shape))
    R = 6.5
    print(f"[gpu] U^dagger V b={b} n={n}", flush=True)
    pat = O.pattern(xyz, R)
    a, x = (rng.uniform(-1, 1, size=(pat.nnzb, b, b)) for _ in range(2))
    ctx = rtdm.Context(0, unit_check_every=2)
    try:
        rtdm.rtdm_set_geometry(ctx.h, xyz, np.full(n, b, dtype=np.int32))
        rtdm.rtdm_set_ranges(ctx.h, 5.0, R, R)
        rtdm.rtdm_upload(ctx.h, "A", a)
        rtdm.rtdm_upload(ctx.h, "X", x)
        rtdm.rtdm_multiply_noalloc(ctx.h, "U", "A", "X", 1, 0)
        got = rtdm.rtdm_download(ctx.h, "U", b)
        ref, _ = O.spgemm(O.BSM(pat, b, a + 0j), O.BSM(pat, b, x + 0j), pat, 1.0, 1, 0)
        assert rel(got, ref.val) <= TOL
    finally:
        ctx.close()
