"""The propagator of enforced time-reversal symmetry, U = P(E2 E1), sums each
element in ascending order of the contraction index at b = 13 and b = 4.

E1 and E2 are the identity plus something small, so the 1 of (E2)_rr (E1)_rr
enters in the middle of a diagonal element's sum, and of the terms after it,
all of one sign, what is below half an ulp of 1 is lost: which terms come
after it shows in the mean of U's diagonal.  Reference: the same sums one
term after the other in ascending order, from the same E (with a fixed H both
half steps have the propagator of an EM step of half the length, bit for bit).

Tolerance.  The kernels take the contraction in groups of 4 blocks, so up to
4 b of an element's N_k terms may change sides: with 1,300 terms and a mean
loss of 1e-15 by less than 4e-17.  A diagonal element's error is that of some
hundreds of roundings of half an ulp below 1 (1.1e-16), 1.6e-15 at most, so
the mean over N > 2,800 of the difference of two orders scatters by 4e-17.
One ulp of 1 (2.2e-16) is more than four times that beside the shift.
"""

import numpy as np
import pytest

from paper_1404_5776_amd import rtdm, synth
from tests._common import gpu_context

pytestmark = pytest.mark.gpu

DT = 0.05


def _dense(blocks, rp, col, n, b):
    out = np.zeros((n, b, n, b))
    out[np.repeat(np.arange(n), np.diff(rp)), :, col, :] = blocks
    return out.reshape(n * b, n * b)


def _u(s, dt, **opts):
    ctx = gpu_context(s, h_model="fixed", **opts)
    rtdm.rtdm_build_inverse(ctx.h)
    rtdm.rtdm_step(ctx.h, dt, 1)
    rp, col = rtdm.rtdm_pattern(ctx.h, "U")
    U = rtdm.rtdm_download(ctx.h, "U", s.b)
    ctx.close()
    return _dense(U.real, rp, col, s.n_atoms, s.b), _dense(U.imag, rp, col, s.n_atoms, s.b)


@pytest.mark.parametrize("b,cells,R", [(13, (3, 3, 3), 12.0), (4, (5, 5, 5), 12.0)])
def test_diagonal_of_u_as_summed_in_ascending_order(b, cells, R):
    s = synth.diamond_lattice(cells, b, 10.0, R, seed=77, k0="local", h_model="fixed")
    N = s.n_atoms * b
    assert N > 2800
    er, ei = _u(s, 0.5 * DT)
    ur, ui = _u(s, DT, propagator="etrs")
    rr, ii = np.zeros(N), np.zeros(N)
    for k in range(N):
        rr += er[:, k] * er[k, :]
        ii += ei[:, k] * ei[k, :]
    err = np.diagonal(ur) - (rr - ii)
    eps = np.finfo(float).eps
    print(f"[gpu] ETRS diagonal b={b} n={s.n_atoms}: mean difference {err.mean():.2e}, rms "
          f"{np.sqrt((err ** 2).mean()):.2e}", flush=True)
    assert abs(err.mean()) <= eps
