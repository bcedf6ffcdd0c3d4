"""Charges taken in the launch that Hermitises K (small systems) against the
launch that reads the finished K.

Both add the same products K_ij[a][c] S_ji[c][a] in the same order and form
K_ij = (Kn_ij + Kn_ji^H) / 2 with the same operations, so the charges agree
bit for bit.  Sizes: one atom, blocks of 1, 4, 5 and 13 functions, pairs of the
overlap outside K's range and K's largest size of one launch (2^20 elements)
and just beyond it.
"""

import numpy as np
import pytest

from paper_1404_5776_amd import rtdm, synth
from tests._common import gpu_context

pytestmark = pytest.mark.gpu


def _system(n, b, R_HS, R_K):
    rng = np.random.default_rng(100 + n)
    xyz = synth.cluster_positions(n, rng) if n > 1 else np.zeros((1, 3))
    return synth.build_system(f"n{n}_b{b}", xyz, b, R_HS, R_K, 7, k0="exact", h_model="mulliken")


# 256 atoms, b = 4, every pair within R_K: 2^20 elements of K; 257 atoms: beyond
@pytest.mark.parametrize("n,b,R_HS,R_K", [(1, 4, 6.0, 8.0), (9, 1, 6.0, 8.0), (9, 5, 8.0, 6.0), (20, 4, 9.0, 5.0),
                                          (17, 13, 8.0, 10.0), (256, 4, 6.0, 400.0), (257, 4, 6.0, 400.0)])
@pytest.mark.parametrize("use_graph", [0, 1])
def test_step_charges_are_those_of_k(n, b, R_HS, R_K, use_graph):
    s = _system(n, b, R_HS, R_K)
    ctx = gpu_context(s, h_model="mulliken", use_graph=use_graph, graph_steps=2)
    try:
        rtdm.rtdm_build_inverse(ctx.h)
        rtdm.rtdm_apply_kick(ctx.h, s.kappa)
        rtdm.rtdm_step(ctx.h, s.dt, 4)
        before = rtdm.rtdm_get_state(ctx.h, n)[2 + n:2 + 2 * n].copy()     # q(t - dt)
        q = rtdm.rtdm_get_state(ctx.h, n)[2:2 + n].copy()
        rtdm.rtdm_step(ctx.h, s.dt, 1)
        assert np.array_equal(rtdm.rtdm_get_state(ctx.h, n)[2 + n:2 + 2 * n], q)
        assert not np.array_equal(before, q) or n == 1
        q = rtdm.rtdm_get_state(ctx.h, n)[2:2 + n].copy()
        K = rtdm.rtdm_download(ctx.h, "K", b)
        rtdm.rtdm_upload(ctx.h, "K", K)                                     # charges from K anew
        rtdm.rtdm_observables(ctx.h)
        assert np.array_equal(rtdm.rtdm_get_state(ctx.h, n)[2:2 + n], q)
    finally:
        ctx.close()
