"""Products on re-laid-out operands against the oracle, element by element.

The b = 13 FP64 row-run products read both operands in pair layout (two
contraction indices per 16-byte load, odd last index alone, lanes past the
13th repeating the 13th).  The systems are the sizes where that can go wrong:
a single atom, a pair, odd row lengths (a run of one output), runs whose
entries do not fill a group of four, atoms without neighbours.

Bound: both sides sum L products of doubles per real component, each with a
forward error of at most L eps sum |a||b|; a complex component holds two real
sums, so |C - C_ref| <= 2 * 2 (L + 2) eps * P(|A||B|) with |.| the largest
component.
"""

import numpy as np
import pytest

from oracle import oracle as O
from paper_1404_5776_amd import rtdm, synth
from tests._common import TOL, rel

pytestmark = pytest.mark.gpu

# (output, left, right, op(left), op(right)) on the kind's ranges
KINDS = {"XH": ("A", "X", "H0", 0, 0), "AT": ("X", "A", "A", 0, 0), "UK": ("W", "U", "K", 0, 0),
         "WU": ("K", "W", "U", 0, 1)}


def _positions(name):
    if name == "one":
        return np.zeros((1, 3))
    if name == "two":
        return np.array([[0.0, 0.0, 0.0], [0.0, 3.1, 0.4]])
    if name == "isolated":
        return np.concatenate([synth.cluster_positions(7, np.random.default_rng(5)),
                               np.array([[100.0, 0.0, 0.0], [0.0, 150.0, 0.0]])])
    return synth.cluster_positions(int(name), np.random.default_rng(int(name)))


def _check(b, xyz, ranges, kind):
    R_HS, R_P, R_K = ranges
    print(f"[gpu] {kind} b={b} n={len(xyz)} ranges={ranges}", flush=True)
    slot_r = {"S": R_HS, "H0": R_HS, "H": R_HS, "X": R_P, "A": R_P, "U": R_P, "K": R_K, "W": R_K}
    out, left, right, op_a, op_b = KINDS[kind]
    ctx = rtdm.Context(0)
    try:
        rtdm.rtdm_set_geometry(ctx.h, xyz, np.full(len(xyz), b, dtype=np.int32))
        rtdm.rtdm_set_ranges(ctx.h, R_HS, R_P, R_K)
        ctx.b = b
        mats, pats = {}, {}
        rng = np.random.default_rng(17)
        for s in (left, right, out):
            pats[s] = O.pattern(xyz, slot_r[s])
        for s in dict.fromkeys((left, right)):
            v = rng.uniform(-1, 1, size=(pats[s].nnzb, b, b))
            if s in "UKW":
                v = v + 1j * rng.uniform(-1, 1, size=v.shape)
            rtdm.rtdm_upload(ctx.h, s, v)
            mats[s] = O.BSM(pats[s], b, v.astype(np.complex128))
        rtdm.rtdm_multiply(ctx.h, out, left, right, op_a, op_b)
        got = rtdm.rtdm_download(ctx.h, out, b)
        ref, _ = O.spgemm(mats[left], mats[right], pats[out], 1.0, op_a, op_b)

        def big(m):
            return O.BSM(m.pat, b, np.maximum(np.abs(m.val.real), np.abs(m.val.imag)).astype(np.complex128))

        mag, _ = O.spgemm(big(mats[left]), big(mats[right]), pats[out], 1.0, op_a, op_b)
        L = b * int(np.diff(pats[left].row_ptr).max())
        bound = 4.0 * (L + 2) * np.finfo(float).eps * mag.val.real
        err = np.abs(got - ref.val)
        assert np.all(err <= bound), (float((err - bound).max()), float(err.max()))
    finally:
        ctx.close()


@pytest.mark.parametrize("kind", sorted(KINDS))
@pytest.mark.parametrize("name", ["one", "two", "isolated", "5", "23", "38"])
def test_pair_layout_b13(name, kind):
    _check(13, _positions(name), (5.0, 8.0, 7.0), kind)


@pytest.mark.parametrize("kind", sorted(KINDS))
@pytest.mark.parametrize("ranges", [(5.0, 6.5, 6.5), (6.5, 6.5, 4.0), (4.0, 5.0, 11.0)])
def test_transposed_right_operand_b4(ranges, kind):
    """b = 4 over enough runs of 16 (at least 4,096) for the kernel that reads
    A by rows and B with transposed blocks, two entries at a time: short rows
    (one partly filled run each), odd numbers of entries, rows of several runs."""
    _check(4, _grid({11.0: 1400}.get(ranges[2], 4200)), ranges, kind)


@pytest.mark.parametrize("kind", ["WU", "UK"])
@pytest.mark.parametrize("n", [1, 2, 33, 64, 330, 900])
def test_split_runs_b4(n, kind):
    """The split form of few runs (8 waves a run below 1,024 runs, 4 below
    4,096): a conjugate-transposed right operand two entries at a time, a plain
    one by rows; runs of fewer pairs of entries than waves."""
    _check(4, _grid(n), (5.0, 9.0, 8.0), kind)


@pytest.mark.parametrize("n", [1, 2, 5, 23])
def test_inverse_iteration_b13(n):
    """The b = 13 iteration that makes X' and both its operand forms in one pass,
    with ranges that keep every pair: X is the inverse of S.  The last step
    forms 2 X - X (S X) with sums of N products each, so its rounding is at
    most 2 (N + 2) eps (1 + |X||S|) |X|; its own error is the square of the
    one before (below 1e-10).   X H0 then reads the same X."""
    b, xyz = 13, synth.cluster_positions(n, np.random.default_rng(n)) if n > 1 else np.zeros((1, 3))
    print(f"[gpu] inverse b={b} n={n}", flush=True)
    R = 200.0
    pat = O.pattern(xyz, R)
    rng = np.random.default_rng(41)
    N = n * b
    off = rng.uniform(-1, 1, size=(N, N))
    S = np.eye(N) + 0.3 / N * (off + off.T)
    blocks = S.reshape(n, b, n, b).transpose(0, 2, 1, 3).reshape(n * n, b, b)
    ctx = rtdm.Context(0)
    try:
        rtdm.rtdm_set_geometry(ctx.h, xyz, np.full(n, b, dtype=np.int32))
        rtdm.rtdm_set_ranges(ctx.h, R, R, R)
        ctx.b = b
        assert pat.nnzb == n * n
        rtdm.rtdm_upload(ctx.h, "S", np.ascontiguousarray(blocks))
        _, res = rtdm.rtdm_build_inverse(ctx.h)
        X = np.real(rtdm.rtdm_download(ctx.h, "X", b)).reshape(n, n, b, b).transpose(0, 2, 1, 3).reshape(N, N)
        want = np.linalg.inv(S)
        nx = np.linalg.norm(want, 2)
        bound = (2.0 * (N + 2) * np.finfo(float).eps * (1.0 + N * nx * np.linalg.norm(S, 2)) + 1e-20) * nx
        assert res < 1e-10
        assert np.linalg.norm(X - want, 2) <= bound, (np.linalg.norm(X - want, 2), bound)
        # the left form of X: X H0 as a product
        H = rng.uniform(-1, 1, size=(n * n, b, b))
        rtdm.rtdm_upload(ctx.h, "H0", H)
        rtdm.rtdm_multiply(ctx.h, "A", "X", "H0", 0, 0)
        A = np.real(rtdm.rtdm_download(ctx.h, "A", b))
        ref, _ = O.spgemm(O.BSM(pat, b, X.reshape(n, b, n, b).transpose(0, 2, 1, 3).reshape(n * n, b, b).astype(complex)),
                          O.BSM(pat, b, H.astype(complex)), pat, 1.0, 0, 0)
        assert np.abs(A - ref.val.real).max() <= 4.0 * (N + 2) * np.finfo(float).eps * N * nx
    finally:
        ctx.close()


@pytest.mark.parametrize("b,n", [(4, 30), (4, 4200), (5, 30), (13, 60)])
def test_inverse_iteration_matches_oracle(b, n):
    """The truncated iteration against the oracle's: at b = 4 with enough runs
    W and X' are written as the transposed blocks that the products read, below
    that (and at other block sizes) by rows.  Same number of iterations; X at
    the 1e-10 relative Frobenius bar of the parity tests."""
    print(f"[gpu] inverse b={b} n={n}", flush=True)
    xyz, (R_HS, R_P, R_K) = _grid(n), (5.0, 6.5, 6.5)
    pat = O.pattern(xyz, R_HS)
    rng = np.random.default_rng(43)
    S = np.zeros((pat.nnzb, b, b))
    row = np.repeat(np.arange(n), np.diff(pat.row_ptr))
    S[:] = 0.01 * rng.uniform(-1, 1, size=S.shape)
    at = {(i, j): p for p, (i, j) in enumerate(zip(row, pat.col))}
    for (i, j), p in at.items():
        if i < j:
            S[at[(j, i)]] = S[p].T
        elif i == j:
            S[p] = np.eye(b) + 0.5 * (S[p] + S[p].T)
    ctx = rtdm.Context(0)
    try:
        rtdm.rtdm_set_geometry(ctx.h, xyz, np.full(n, b, dtype=np.int32))
        rtdm.rtdm_set_ranges(ctx.h, R_HS, R_P, R_K)
        rtdm.rtdm_upload(ctx.h, "S", S)
        it, _ = rtdm.rtdm_build_inverse(ctx.h)
        X = rtdm.rtdm_download(ctx.h, "X", b)
        ref = O.hotelling(O.BSM(pat, b, S.astype(np.complex128)), O.pattern(xyz, R_P))
        assert it == ref.iters
        assert rel(X, ref.X.val) <= TOL
    finally:
        ctx.close()


@pytest.mark.parametrize("b,n", [(4, 4200), (13, 300)])
def test_products_issued_on_two_streams(b, n):
    """Two products of one context that share no slot, on two streams without
    an order of the caller's: both lay their right operand out in the same
    buffer, so the library orders them; bytes as when issued one by one."""
    import torch

    xyz, (R_HS, R_P, R_K) = _grid(n), (5.0, 6.5, 6.5)
    slot_r = {"S": R_HS, "X": R_P, "U": R_P, "K": R_K}
    ctx = rtdm.Context(0)
    try:
        rtdm.rtdm_set_geometry(ctx.h, xyz, np.full(n, b, dtype=np.int32))
        rtdm.rtdm_set_ranges(ctx.h, R_HS, R_P, R_K)
        rng = np.random.default_rng(23)
        for m in ("S", "X", "U", "K"):
            v = rng.uniform(-1, 1, size=(O.pattern(xyz, slot_r[m]).nnzb, b, b))
            rtdm.rtdm_upload(ctx.h, m, v + 1j * v[::-1] if m in "UK" else v)
        jobs = [("A", "S", "X"), ("W", "U", "K")]      # the kinds S X and U K
        ref = []
        for j in jobs:
            rtdm.rtdm_multiply(ctx.h, *j, 0, 0)
            torch.cuda.synchronize()
            ref.append(rtdm.rtdm_download(ctx.h, j[0], b))
        streams = [torch.cuda.Stream() for _ in jobs]
        for rep in range(8):
            print(f"[gpu] two streams b={b} n={n} rep={rep}", flush=True)
            for _ in range(4):
                for j, st in zip(jobs, streams):
                    rtdm.rtdm_multiply(ctx.h, *j, 0, 0, 1.0, st)
            torch.cuda.synchronize()
            for j, r in zip(jobs, ref):
                assert np.array_equal(rtdm.rtdm_download(ctx.h, j[0], b), r), (j, rep)
    finally:
        ctx.close()


def _grid(n):
    rng = np.random.default_rng(3)
    g = DENSITY ** (-1.0 / 3.0)
    m = int(np.ceil(n ** (1.0 / 3.0)))
    p = np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing="ij"), -1).reshape(-1, 3)[:n] * g
    return np.ascontiguousarray(p + rng.uniform(-0.4, 0.4, size=p.shape))


DENSITY = synth.CLUSTER_DENSITY
