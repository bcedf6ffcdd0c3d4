"""The propagator of enforced time-reversal symmetry, U = P(E2 E1), has no
systematic error on its diagonal.

E1 and E2 are the identity plus something small.  In the plain product the 1
of (E2)_rr (E1)_rr enters somewhere in the middle of a sum of a thousand terms
of one sign, and those after it that are below half an ulp of 1 are lost, all
to the same side.  Reference: the same U minus the identity, D2 + D1 + P(D2 D1)
with D = E - 1, in which every sum is small.  Each diagonal element of the
library's U is 1 plus sums of that size, rounded at most 2 p + 2 times to half
an ulp of 1 (the Taylor sums of E1 and E2, the last sum), to either side; the
mean over N elements is then below half an ulp: (2 p + 2) / sqrt(N) < 1 at
N > 144, p = 5.
"""

import numpy as np
import pytest

from paper_1404_5776_amd import rtdm, synth
from tests._common import gpu_context

pytestmark = pytest.mark.gpu


def _dense(blocks, rp, col, n, b):
    out = np.zeros((n, b, n, b))
    out[np.repeat(np.arange(n), np.diff(rp)), :, col, :] = blocks
    return out.reshape(n * b, n * b)


@pytest.mark.parametrize("b,cells,R", [(13, (3, 3, 3), 12.0), (4, (6, 6, 6), 12.0)])
def test_no_bias_on_the_diagonal_of_u(b, cells, R):
    s = synth.diamond_lattice(cells, b, 10.0, R, seed=77, k0="local", h_model="fixed")
    n, dt, p = s.n_atoms, 0.05, 5
    ctx = gpu_context(s, h_model="fixed", propagator="etrs")
    rtdm.rtdm_build_inverse(ctx.h)
    rtdm.rtdm_step(ctx.h, dt, 1)
    rp, col = rtdm.rtdm_pattern(ctx.h, "U")
    U = rtdm.rtdm_download(ctx.h, "U", b)
    A = _dense(np.real(rtdm.rtdm_download(ctx.h, "A", b)), rp, col, n, b)
    ctx.close()
    mask = _dense(np.ones((col.size, b, b)), rp, col, n, b)
    # D = E - 1 of exp(-i dt/2 A), order p, every power truncated (a fixed H: E1 = E2)
    re, im, t = np.zeros_like(A), np.zeros_like(A), 0.5 * dt * A
    im -= t
    for k in range(2, p + 1):
        t = (A @ t) * mask * (0.5 * dt / k)
        if k % 2 == 0:
            re += t if k % 4 == 0 else -t
        else:
            im += t if k % 4 == 3 else -t
    ref = 2.0 * re + (re @ re - im @ im) * mask
    got = _dense(U.real, rp, col, n, b)
    err = (np.diagonal(got) - 1.0) - np.diagonal(ref)
    eps = np.finfo(float).eps
    N = n * b
    assert N > 144
    print(f"[gpu] ETRS diagonal b={b} n={n}: mean error {err.mean():.2e}, largest {np.abs(err).max():.2e}", flush=True)
    assert abs(err.mean()) <= eps / 2
    # every element: the roundings at 1, and the sums of small terms (N terms, each below |D|_rk |D|_kr)
    small = N * eps * ((np.abs(re) + np.abs(im)) @ (np.abs(re) + np.abs(im))).diagonal()
    assert np.all(np.abs(err) <= (2 * p + 2) * eps / 2 + small)
