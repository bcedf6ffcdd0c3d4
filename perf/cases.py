"""Performance cases of the library: the calls a propagation program makes.

Each case is one kind of program over the size ranges of the workloads of
`synth.py` and `bench.py` (clusters of 4 or 13 functions per atom with cut-offs
8 / 12 bohr, diamond-like lattices with 10 / 8, 12 or 16 bohr):

  propagate  a K of the ground state is uploaded, kicked, stepped, and the
             observable trace and the final K are read back (rtdm_upload,
             rtdm_apply_kick, rtdm_step, rtdm_dipole_trace, rtdm_download);
  batch      clusters of both block sizes with their x, y and z kicks advanced
             together by one captured graph (rtdm_batch_step), every kick
             set's group traces and K read back;
  inverse    the truncated inverse of a new overlap matrix (rtdm_upload of S,
             rtdm_build_inverse, rtdm_download of X);
  mlp        prediction, loss and gradient of the network that starts the
             inverse from a learned guess (rtdm_mlp_predict, rtdm_mlp_loss_grad).

What a program prepares once (geometry, cut-offs, S, H0, the inverse, the
batch, the network's weights) is made by prepare().  Inputs follow the recipe
of synth.py (unit diagonal overlap, Gaussian-decaying random off-diagonal
blocks, a gapped on-site Hamiltonian); K is a stand-in of a gapped density
matrix: occupied diagonal and exponentially decaying off-diagonal blocks.
"""

import math

import numpy as np
import torch

from paper_1404_5776_amd import rtdm

DEV = "cuda:0"
NN = 3.37            # nearest-neighbour distance of the lattice, decay length of S and H0 (bohr)
DENSITY = 0.026      # atoms per cubic bohr of a cluster
HIDDEN = 128         # width of the learned start's network


def _step_case(name, **kw):
    c = {"name": name, "kind": "propagate", "geometry": "lattice", "nx": 0, "ny": 0, "nz": 0, "atoms": 0, "b": 4,
         "r_hs": 10.0, "r_k": 12.0, "model": "mulliken", "propagator": "em", "precision": "fp64", "graph": False,
         "field": False, "corrector": 0, "unit_every": 0, "steps": 1, "dt": 0.05}
    c.update(kw)
    return c


def listed():
    return [
        # The smallest call: one step of a molecule-sized cluster, read back at
        # once, as a program that couples every step to other code does.
        _step_case("cluster20_b4_step", geometry="cluster", atoms=20, r_hs=8.0, model="fixed", steps=1),
        # The 64-atom cluster of the tests and of `bench.py --leg small`: a
        # hundred short steps, where launches and latencies count.
        _step_case("cluster64_b4_100steps", geometry="cluster", atoms=64, r_hs=8.0, model="fixed", steps=100),
        # The 64-cluster workload in small: clusters of both block sizes, x/y/z
        # kicks, one captured graph of 16 steps (and 4 steps beyond it).
        {"name": "batch12_kicksets", "kind": "batch", "clusters4": 7, "clusters13": 5, "smallest": 50, "largest": 400,
         "steps": 20, "graph_steps": 16, "dt": 0.05},
        # A 512-atom lattice of 13 functions, H following the charges, steps
        # replayed from graphs.
        _step_case("lattice512_b13_graph", nx=4, ny=4, nz=4, b=13, r_k=16.0, graph=True, steps=4),
        # The headline workload of bench.py at full size: 4,096 atoms of 13
        # functions, R_K 16.
        _step_case("lattice4096_b13", nx=8, ny=8, nz=8, b=13, r_k=16.0, steps=1),
        # The 32,768-atom lattice of 4 functions at the middle of its cut-off sweep.
        _step_case("lattice32768_b4_rk12", nx=16, ny=16, nz=16, r_k=12.0, steps=2),
        # The shortest cut-off of that sweep on an odd-shaped lattice: K on a
        # smaller range than H, S and U.
        _step_case("lattice7560_b4_rk8", nx=9, ny=7, nz=15, r_k=8.0, steps=5),
        # The reduced-precision option that production runs at b = 4 take (late
        # Taylor terms in FP32), long cut-off, with the unitarity monitor.
        _step_case("lattice2744_b4_rk16_fp32taylor", nx=7, ny=7, nz=7, r_k=16.0, precision="fp32_taylor", steps=4,
                   unit_every=4),
        # Enforced time-reversal symmetry with self-consistent corrector passes
        # right after the kick, 13 functions per atom.
        _step_case("lattice360_b13_etrs_corrector", nx=3, ny=5, nz=3, b=13, r_k=12.0, propagator="etrs", corrector=2,
                   steps=3),
        # Fourth-order Magnus under a Gaussian field.
        _step_case("lattice1728_b4_m4_field", nx=6, ny=6, nz=6, r_k=12.0, propagator="m4", field=True, steps=3),
        # The inverse of a new overlap matrix, 13 functions, as every geometry needs it once.
        {"name": "inverse1000_b13", "kind": "inverse", "geometry": "lattice", "nx": 5, "ny": 5, "nz": 5, "atoms": 0,
         "b": 13, "r_hs": 10.0, "r_k": 16.0},
        # Forward and backward of the learned start's network on a training batch.
        {"name": "mlp4096_b4", "kind": "mlp", "b": 4, "samples": 4096},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _cells(rng, lo, hi):
    """A lattice of about lo to hi atoms (8 per cell), sides of unlike length."""
    n = max(1.0, _log_int(rng, lo, hi) / 8.0)
    nx = max(1, int(round(n ** (1.0 / 3.0) * rng.uniform(0.75, 1.3))))
    ny = max(1, int(round(math.sqrt(n / nx) * rng.uniform(0.85, 1.15))))
    nz = max(1, int(n / (nx * ny)))
    return nx, ny, nz


def draw(rng):
    kind = rng.choice(["cluster", "cluster", "lattice4", "lattice4", "lattice4", "lattice13", "lattice13", "batch",
                       "inverse", "mlp"])
    if kind == "cluster":
        b = rng.choice([4, 13])
        atoms = _log_int(rng, 12, 900 if b == 4 else 300)
        c = _step_case("", geometry="cluster", atoms=atoms, b=b, r_hs=8.0, r_k=12.0,
                       model=rng.choice(["fixed", "mulliken"]), graph=rng.random() < 0.4, steps=_log_int(rng, 1, 40))
    elif kind == "lattice4":
        r_k = rng.choice([8.0, 12.0, 12.0, 16.0])
        nx, ny, nz = _cells(rng, 64, {8.0: 30000, 12.0: 24000, 16.0: 6000}[r_k])
        precision = rng.choice(["fp64", "fp64", "fp64", "fp32_taylor", "bf16x3_taylor"])
        prop = rng.choice(["em", "em", "em", "etrs", "m4"]) if precision == "fp64" and nx * ny * nz <= 500 else "em"
        c = _step_case("", nx=nx, ny=ny, nz=nz, r_k=r_k, precision=precision, propagator=prop,
                       field=prop != "em" and rng.random() < 0.5, graph=rng.random() < 0.3, steps=rng.randint(1, 2))
    elif kind == "lattice13":
        r_k = rng.choice([12.0, 16.0])
        prop = rng.choice(["em", "em", "etrs", "m4"])
        nx, ny, nz = _cells(rng, 32, 2400 if prop == "em" else 400)
        c = _step_case("", nx=nx, ny=ny, nz=nz, b=13, r_k=r_k, propagator=prop, graph=rng.random() < 0.3, steps=1)
    elif kind == "batch":
        c = {"kind": "batch", "clusters4": rng.randint(2, 8), "clusters13": rng.randint(2, 5),
             "smallest": rng.randint(20, 60), "largest": _log_int(rng, 80, 400), "steps": rng.randint(4, 20),
             "graph_steps": rng.choice([4, 8, 16]), "dt": 0.05}
    elif kind == "inverse":
        b = rng.choice([4, 13])
        nx, ny, nz = _cells(rng, 64, 12000 if b == 4 else 1500)
        c = {"kind": "inverse", "geometry": "lattice", "nx": nx, "ny": ny, "nz": nz, "atoms": 0, "b": b, "r_hs": 10.0,
             "r_k": rng.choice([8.0, 12.0, 16.0]) if b == 4 and nx * ny * nz < 800 else 12.0}
    else:
        c = {"kind": "mlp", "b": rng.choice([4, 4, 13]), "samples": _log_int(rng, 33, 6000)}
    c.pop("name", None)
    return c


# ------------------------------------------------------------------ inputs

def _morton(xyz):
    """Atoms in Z-curve order of an NN grid, as the generators of the workloads emit them."""
    cell = np.floor((xyz - xyz.min(axis=0)) / NN).astype(np.int64)
    key = np.zeros(len(xyz), dtype=np.int64)
    for bit in range(12):
        for ax in range(3):
            key |= ((cell[:, ax] >> bit) & 1) << (3 * bit + ax)
    return np.ascontiguousarray(xyz[np.argsort(key, kind="stable")])


def _cluster(n, rng):
    """n atoms at a cluster's density, at least 2.5 bohr apart: a jittered grid, the corner farthest out left off."""
    g = DENSITY ** (-1.0 / 3.0)
    m = math.ceil(n ** (1.0 / 3.0))
    p = np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing="ij"), -1).reshape(-1, 3).astype(np.float64)
    p = p[np.argsort(p.sum(axis=1), kind="stable")[:n]]
    return _morton(g * p + rng.uniform(-0.5, 0.5, size=(n, 3)) * (g - 2.5))


def _positions(case):
    """The atoms of a case: one geometry, whose S, H0 and K the seed draws."""
    rng = np.random.default_rng(17 + 8 * (case["atoms"] + case["nx"]) + case["b"])
    if case["geometry"] == "cluster":
        return _cluster(case["atoms"], rng)
    a = 4.0 * NN / math.sqrt(3.0)
    basis = np.array([[0, 0, 0], [0, .5, .5], [.5, 0, .5], [.5, .5, 0],
                      [.25, .25, .25], [.25, .75, .75], [.75, .25, .75], [.75, .75, .25]])
    g = np.stack(np.meshgrid(np.arange(case["nx"]), np.arange(case["ny"]), np.arange(case["nz"]), indexing="ij"), -1)
    xyz = (g.reshape(-1, 1, 3) + basis.reshape(1, 8, 3)).reshape(-1, 3) * a
    return _morton(xyz + rng.normal(0.0, 0.02 * NN, size=xyz.shape))


def _pairs(x, R):
    """(rows, cols, d) of the pairs closer than R and the diagonal, row by row, columns ascending."""
    n = x.shape[0]
    rows, cols, d2s = [], [], []
    step = max(1, (1 << 26) // n)
    for i0 in range(0, n, step):
        xi = x[i0:i0 + step]
        d2 = torch.zeros(xi.shape[0], n, dtype=torch.float64, device=x.device)
        for k in range(3):
            t = xi[:, k:k + 1] - x[None, :, k]
            d2 += t * t
        i, j = torch.nonzero(d2 < R * R, as_tuple=True)
        rows.append(i + i0)
        cols.append(j)
        d2s.append(d2[i, j])
    return torch.cat(rows), torch.cat(cols), torch.cat(d2s).sqrt()


def _symmetric(rows, cols, n, b, gen):
    """Uniform (-1, 1) blocks, block (j, i) the transpose of block (i, j)."""
    u = torch.rand(rows.numel(), b, b, dtype=torch.float64, device=rows.device, generator=gen).mul_(2.0).sub_(1.0)
    key = rows * n + cols
    tr = torch.searchsorted(key, cols * n + rows)
    low = rows > cols
    u[low] = u[tr[low]].transpose(1, 2)
    dg = torch.nonzero(rows == cols).flatten()
    u[dg] = 0.5 * (u[dg] + u[dg].transpose(1, 2))
    return u, dg


def _matrices(x, b, r_hs, r_k, seed):
    """(pattern of S and H0, S, H0, pattern of K, K) as blocks in pattern order."""
    n = x.shape[0]
    gen = torch.Generator(device=x.device).manual_seed(7919 * seed + 11)
    rows, cols, d = _pairs(x, r_hs)
    decay = torch.exp(-(d / NN) ** 2)[:, None, None]
    S, dg = _symmetric(rows, cols, n, b, gen)
    S *= decay
    S[dg] = 0.0
    rs = torch.segment_reduce(S.abs().sum(2), "sum", lengths=torch.bincount(rows, minlength=n), axis=0)
    S *= 0.8 / max(float(rs.max()), 1e-300)
    S[dg] = torch.eye(b, dtype=torch.float64, device=x.device)
    H, _ = _symmetric(rows, cols, n, b, gen)
    level = torch.where(torch.arange(b, device=x.device) < b // 2, -0.5, 0.5).double()
    noise = H[dg] * 0.05
    H *= -0.05 * decay
    H[dg] = torch.diag(level) + noise
    krows, kcols, kd = _pairs(x, r_k)
    K, kdg = _symmetric(krows, kcols, n, b, gen)
    K *= 0.05 * torch.exp(-kd / 3.0)[:, None, None]
    K[kdg] += torch.diag((torch.arange(b, device=x.device) < b // 2).double())
    return (rows, cols), S, H, (krows, kcols), K


def _load(ctx, xyz, x, b, r_hs, r_k, seed, groups=None):
    """The set-up calls of a program, with S, H0 and K handed over in device memory; returns its S and the K it starts from."""
    n = xyz.shape[0]
    rtdm.rtdm_set_geometry(ctx.h, xyz, np.full(n, b, dtype=np.int32))
    rtdm.rtdm_set_ranges(ctx.h, r_hs, max(r_hs, r_k), r_k)
    if groups is not None:
        rtdm.rtdm_set_groups(ctx.h, groups)
    ps, S, H, pk, K = _matrices(x, b, r_hs, r_k, seed)
    for slot, (rows, cols) in (("S", ps), ("K", pk)):
        rp, col = rtdm.rtdm_pattern(ctx.h, slot)
        if col.size != cols.numel() or not np.array_equal(col, cols.cpu().numpy()):
            raise RuntimeError("the generated pattern of %s is not the library's" % slot)
    rtdm.rtdm_upload(ctx.h, "S", S)
    rtdm.rtdm_upload(ctx.h, "H0", H)
    rtdm.rtdm_upload(ctx.h, "K", K)
    return S, K


class _Batch:
    """A batch handle that is given back before the contexts it steps."""

    def __init__(self, ctxs, graph_steps):
        self.ctxs = ctxs
        self.h = rtdm.rtdm_batch_create([c.h for c in ctxs], graph_steps=graph_steps)

    def __del__(self):
        rtdm.rtdm_batch_destroy(self.h)


def _kappa(seed):
    """A kick of 0.01 per bohr along one axis."""
    k = [0.0, 0.0, 0.0]
    k[seed % 3] = 0.01
    return k


FIELD_E0, FIELD_T0, FIELD_SIGMA = (0.002, -0.001, 0.0015), 0.08, 0.06


def _batch_members(case):
    """Per block size: positions of its clusters laid out along x beyond every range, and the group pointer."""
    rng = np.random.default_rng(29 + case["smallest"])
    out = []
    for b, m in ((4, case["clusters4"]), (13, case["clusters13"])):
        lo, hi = math.log(case["smallest"]), math.log(case["largest"])
        parts, ptr, x0 = [], [0], 0.0
        for k in range(m):                      # sizes log-uniform over the range, larger blocks on fewer atoms
            n = int(math.exp(lo + (hi - lo) * (k + 0.5) / m))
            p = _cluster(max(8, n if b == 4 else n // 2), rng)
            p[:, 0] += x0 - p[:, 0].min()
            x0 = p[:, 0].max() + 25.0
            parts.append(p)
            ptr.append(ptr[-1] + len(p))
        out.append((b, np.ascontiguousarray(np.concatenate(parts)), np.asarray(ptr, dtype=np.int64)))
    return out


KICKS = ((0.01, 0.0, 0.0), (0.0, 0.01, 0.0), (0.0, 0.0, 0.01))


def _mlp_inputs(case, seed):
    b, n = case["b"], case["samples"]
    rng = np.random.default_rng(1000003 * seed + 31)
    v = rng.normal(size=(n, 3))
    v *= (rng.uniform(0.3, 1.0, size=(n, 1)) / np.linalg.norm(v, axis=1, keepdims=True))
    r = np.linalg.norm(v, axis=1, keepdims=True)
    s = 0.1 * np.exp(-(10.0 * r / NN) ** 2) * rng.uniform(-1.0, 1.0, size=(n, b * b))
    desc = np.concatenate([v, r, s], axis=1).astype(np.float32)
    target = (0.02 * np.exp(-5.0 * r) * rng.uniform(-1.0, 1.0, size=(n, b * b))).astype(np.float32)
    n_in, n_out = 4 + b * b, b * b
    w = np.concatenate([rng.normal(0.0, 1.0 / math.sqrt(n_in), HIDDEN * n_in), rng.normal(0.0, 0.1, HIDDEN),
                        rng.normal(0.0, 0.1 / math.sqrt(HIDDEN), n_out * HIDDEN), rng.normal(0.0, 0.01, n_out)])
    return desc, target, w.astype(np.float32)


def prepare(case, seed):
    if case["kind"] == "mlp":
        desc, target, w = _mlp_inputs(case, seed)
        ctx = rtdm.Context(0)
        rtdm.rtdm_set_geometry(ctx.h, np.zeros((1, 3)), np.full(1, case["b"], dtype=np.int32))
        rtdm.rtdm_mlp_init(ctx.h, seed)
        rtdm.rtdm_mlp_set_weights(ctx.h, w)
        return {"kind": "mlp", "ctx": ctx, "desc": desc, "target": target}
    if case["kind"] == "batch":
        st = {"kind": "batch", "ctx": [], "K": [], "out": [], "groups": [], "steps": case["steps"], "dt": case["dt"]}
        for b, xyz, ptr in _batch_members(case):
            ctx = rtdm.Context(0, n_kicks=3, use_graph=1)
            x = torch.from_numpy(xyz).to(DEV)
            st["K"].append(_load(ctx, xyz, x, b, 8.0, 12.0, seed + b, ptr)[1])
            rtdm.rtdm_build_inverse(ctx.h)
            st["ctx"].append(ctx)
            st["groups"].append(len(ptr) - 1)
            st["out"].append([torch.empty(st["K"][-1].shape, dtype=torch.complex128, device=DEV) for _ in KICKS])
        st["batch"] = _Batch(st["ctx"], case["graph_steps"])
        return st
    xyz = _positions(case)
    x = torch.from_numpy(xyz).to(DEV)
    if case["kind"] == "inverse":
        ctx = rtdm.Context(0)
        S, _ = _load(ctx, xyz, x, case["b"], case["r_hs"], case["r_k"], seed)
        n_x = rtdm.rtdm_pattern(ctx.h, "X")[1].size
        return {"kind": "inverse", "ctx": ctx, "S": S,
                "X": torch.empty(n_x, case["b"], case["b"], dtype=torch.complex128, device=DEV)}
    opts = {"h_model": case["model"], "propagator": case["propagator"], "precision": case["precision"],
            "use_graph": int(case["graph"]), "unit_check_every": case["unit_every"]}
    if case["corrector"]:
        opts.update(sc_steps=case["corrector"], sc_iters=2)
    ctx = rtdm.Context(0, **opts)
    _, K = _load(ctx, xyz, x, case["b"], case["r_hs"], case["r_k"], seed)
    rtdm.rtdm_build_inverse(ctx.h)
    if case["field"]:
        rtdm.rtdm_set_field(ctx.h, FIELD_E0, FIELD_T0, FIELD_SIGMA)
    return {"kind": "propagate", "ctx": ctx, "K": K, "kappa": _kappa(seed), "steps": case["steps"], "dt": case["dt"],
            "out": torch.empty(K.shape, dtype=torch.complex128, device=DEV)}


# ------------------------------------------------------------------ one pass

def run(state):
    if state["kind"] == "mlp":
        h = state["ctx"].h
        y = rtdm.rtdm_mlp_predict(h, state["desc"])
        loss, grad = rtdm.rtdm_mlp_loss_grad(h, state["desc"], state["target"])
        return {"y": y, "loss": loss, "grad": grad}
    if state["kind"] == "inverse":
        h = state["ctx"].h
        rtdm.rtdm_upload(h, "S", state["S"])
        iters, _ = rtdm.rtdm_build_inverse(h)
        rtdm.rtdm_download(h, "X", state["X"].shape[1], out=state["X"])
        return {"iterations": iters, "X": state["X"]}
    if state["kind"] == "batch":
        for ctx, K in zip(state["ctx"], state["K"]):
            rtdm.rtdm_upload(ctx.h, "K", K)
            rtdm.rtdm_apply_kicks(ctx.h, KICKS)
        rtdm.rtdm_batch_step(state["batch"].h, state["dt"], state["steps"])
        res = {}
        for ctx, K, groups, outs in zip(state["ctx"], state["K"], state["groups"], state["out"]):
            b = K.shape[1]
            for k, out in enumerate(outs):
                rtdm.rtdm_select_kick(ctx.h, k)
                res["trace%d_%d" % (b, k)] = rtdm.rtdm_group_trace(ctx.h, groups)
                rtdm.rtdm_download(ctx.h, "K", b, out=out)
                res["K%d_%d" % (b, k)] = out
        return res
    h = state["ctx"].h
    rtdm.rtdm_upload(h, "K", state["K"])
    rtdm.rtdm_apply_kick(h, state["kappa"])
    rtdm.rtdm_step(h, state["dt"], state["steps"])
    trace = rtdm.rtdm_dipole_trace(h)
    rtdm.rtdm_download(h, "K", state["out"].shape[1], out=state["out"])
    return {"trace": trace, "K": state["out"]}


# ------------------------------------------------------------------ work

def _counts(xyz, radii):
    """Stored blocks of each range, and of the block products C = P(A B) for ranges (a, b, c), from up to 192 sampled rows."""
    n = len(xyz)
    rows = np.linspace(0, n - 1, min(n, 192)).astype(int)
    blocks = {r: 0.0 for r in radii}
    prods = {(a, b, c): 0.0 for a in radii for b in radii for c in radii}
    rmax = max(radii)
    for i in rows:
        d2 = ((xyz - xyz[i]) ** 2).sum(axis=1)
        near = np.nonzero(d2 < rmax * rmax)[0]
        di = d2[near]
        x = xyz[near]
        dd = ((x[:, None, :] - x[None, :, :]) ** 2).sum(axis=2)
        for r in radii:
            blocks[r] += float((di < r * r).sum())
        for a, b, c in prods:
            prods[a, b, c] += float((dd[np.ix_(di < a * a, di < c * c)] < b * b).sum())
    f = n / len(rows)
    return {r: v * f for r, v in blocks.items()}, {k: v * f for k, v in prods.items()}


def _step_work(xyz, b, r_hs, r_k, steps, model="fixed", propagator="em", passes=0, kicks=1, field=False, every=0):
    r_p = max(r_hs, r_k)
    nb, T = _counts(xyz, sorted({r_hs, r_k, r_p}))
    rr = 2.0 * b ** 3                                        # flops of one real block product
    xh, at = rr * T[r_p, r_hs, r_p], rr * T[r_p, r_p, r_p]
    uk, wu = 4 * rr * T[r_p, r_k, r_k], 4 * rr * T[r_k, r_p, r_k]
    points = 1 if propagator == "em" else 2
    if propagator == "em":
        u = 4 * at
    elif propagator == "etrs":
        u = 8 * at + 4 * at
    else:
        u = 2 * at + 4 * 4 * at
    # a fixed H: one propagator in all; the on-site model scales columns of X instead of a product per time point
    builds = (steps + passes) if (model == "mulliken" or field) else 1
    flops = (builds if field else 1) * points * xh + builds * u + (steps + passes) * kicks * (uk + wu)
    if every:
        flops += (steps // every) * (2 * rr * T[r_hs, r_p, r_p] + 4 * at)
    e = 8.0 * b * b
    return {"bytes": e * (2 * nb[r_hs] + nb[r_p] + kicks * 4 * nb[r_k]), "flops": flops}


def work(case):
    b = case.get("b")
    if case["kind"] == "mlp":
        n, n_in, n_out = case["samples"], 4 + b * b, b * b
        fwd = 2.0 * n * HIDDEN * (n_in + n_out)
        return {"bytes": 4.0 * n * (2 * n_in + 2 * n_out) + 8.0 * HIDDEN * (n_in + n_out),
                "flops": 2 * fwd + fwd + 2.0 * n * HIDDEN * n_out}
    if case["kind"] == "batch":
        w = {"bytes": 0.0, "flops": 0.0}
        for bb, xyz, _ in _batch_members(case):
            for k, v in _step_work(xyz, bb, 8.0, 12.0, case["steps"], kicks=3).items():
                w[k] += v
        return w
    xyz = _positions(case)
    if case["kind"] == "inverse":
        r_p = max(case["r_hs"], case["r_k"])
        nb, T = _counts(xyz, sorted({case["r_hs"], r_p}))
        iters = 6                                            # to a residual of 1e-10 from the block-Jacobi start
        return {"bytes": 8.0 * b * b * (nb[case["r_hs"]] + nb[r_p]),
                "flops": iters * 2.0 * b ** 3 * (T[case["r_hs"], r_p, r_p] + T[r_p, r_p, r_p])}
    passes = min(case["corrector"], case["steps"]) * 2
    return _step_work(xyz, b, case["r_hs"], case["r_k"], case["steps"], case["model"], case["propagator"], passes,
                      field=case["field"], every=case["unit_every"])


# ------------------------------------------------------------------ 64-bit reference

class _Dense:
    """The truncated algebra on dense matrices: every product is masked to its range."""

    def __init__(self, x, b, r_hs, r_k, seed):
        self.n, self.b = x.shape[0], b
        self.x = x
        (rows, cols), S, H, (kr, kc), K = _matrices(x, b, r_hs, r_k, seed)
        self.krows, self.kcols = kr, kc
        self.S, self.H0, self.K0 = self.dense(rows, cols, S), self.dense(rows, cols, H), self.dense(kr, kc, K)
        self.mk = self.mask(kr, kc)
        if r_k >= r_hs:
            self.prows, self.pcols, self.mp = kr, kc, self.mk
        else:
            self.prows, self.pcols, self.mp = rows, cols, self.mask(rows, cols)

    def dense(self, rows, cols, blocks):
        out = torch.zeros(self.n, self.n, self.b, self.b, dtype=blocks.dtype, device=blocks.device)
        out[rows, cols] = blocks
        return out.permute(0, 2, 1, 3).reshape(self.n * self.b, self.n * self.b)

    def mask(self, rows, cols):
        m = torch.zeros(self.n, self.n, dtype=torch.float64, device=rows.device)
        m[rows, cols] = 1.0
        return m.repeat_interleave(self.b, 0).repeat_interleave(self.b, 1)

    def blocks(self, M, rows, cols):
        return M.view(self.n, self.b, self.n, self.b)[rows, :, cols, :]

    def p(self, M):
        return M * self.mp

    def inverse(self):
        n, b = self.n, self.b
        i = torch.arange(n, device=self.x.device)
        D = torch.linalg.inv(self.S.view(n, b, n, b)[i, :, i, :])
        X = self.dense(i, i, D)
        last = math.inf
        for k in range(50):
            Y = 2.0 * X - self.p(X @ self.p(self.S @ X))
            r = float((Y - X).norm() / Y.norm())
            if not math.isfinite(r) or (k >= 1 and r > last):
                raise RuntimeError("the inverse iteration diverged")
            X, last = Y, r
            if r <= 1e-10:
                return X, k + 1
        raise RuntimeError("the inverse iteration did not converge")

    def charges(self, K):
        return (K.real * self.S.T).sum(dim=1).view(self.n, self.b).sum(dim=1)

    def kick(self, kappa):
        ph = self.x @ torch.tensor(kappa, dtype=torch.float64, device=self.x.device)
        f = torch.polar(torch.ones_like(ph), ph).repeat_interleave(self.b)
        return f[:, None] * self.K0 * f.conj()[None, :]

    def taylor(self, A, dt, p=5):
        U = torch.eye(A.shape[0], dtype=torch.complex128, device=A.device)
        re, im = torch.eye(A.shape[0], dtype=torch.float64, device=A.device), torch.zeros_like(A)
        t = dt * A
        im -= t
        for k in range(2, p + 1):
            t = self.p(A @ t) * (dt / k)
            if k % 2:
                im += t if k % 4 == 3 else -t
            else:
                re += t if k % 4 == 0 else -t
        return torch.complex(re, im)


def _cmm(a, b):
    """Product of complex matrices from real ones."""
    re = a.real.contiguous() @ b.real.contiguous() - a.imag.contiguous() @ b.imag.contiguous()
    im = a.real.contiguous() @ b.imag.contiguous() + a.imag.contiguous() @ b.real.contiguous()
    return torch.complex(re, im)


def _exact_steps(m, case, kappa):
    """(trace rows, K) of the steps of a case on dense matrices."""
    X, _ = m.inverse()
    dt, n, b = case["dt"], m.n, m.b
    K = m.kick(kappa)
    q_ref = m.charges(m.K0)
    q = m.charges(K)
    q_prev = q
    d = m.x - m.x.mean(dim=0)
    half = d.repeat_interleave(b, 0)
    mull = case["model"] == "mulliken"

    def a_of(theta, t, base, qx, qy):
        H = m.H0
        if mull:
            H = H + torch.diag((0.5 * (base + theta * (qx - qy) - q_ref)).repeat_interleave(b))
        if case["field"]:
            f = math.exp(-((t + theta * dt - FIELD_T0) ** 2) / (2.0 * FIELD_SIGMA ** 2))
            v = half @ torch.tensor(FIELD_E0, dtype=torch.float64, device=half.device) * f
            H = H + 0.5 * (v[:, None] + v[None, :]) * m.S
        return m.p(X @ H)

    def build(t, base, qx, qy):
        if case["propagator"] == "em":
            return m.taylor(a_of(0.5, t, base, qx, qy), dt)
        if case["propagator"] == "etrs":
            E1 = m.taylor(a_of(0.0, t, base, qx, qy), 0.5 * dt)
            return m.p(_cmm(m.taylor(a_of(1.0, t, base, qx, qy), 0.5 * dt), E1))
        g = math.sqrt(3.0) / 6.0
        A1, A2 = a_of(0.5 - g, t, base, qx, qy), a_of(0.5 + g, t, base, qx, qy)
        M = torch.complex(-(math.sqrt(3.0) * dt * dt / 12.0) * (m.p(A2 @ A1) - m.p(A1 @ A2)), -0.5 * dt * (A1 + A2))
        U = torch.eye(M.shape[0], dtype=torch.complex128, device=M.device) + M
        T = M
        for k in range(2, 6):
            T = m.p(_cmm(M, T)) / k
            U += T
        return U

    rows, U = [], None
    varies = mull or case["field"]
    for s in range(case["steps"]):
        t = s * dt
        K_new, q_next = None, None
        for it in range(3 if varies and s < case["corrector"] else 1):
            if varies or U is None:
                U = build(t, q, q, q_prev) if it == 0 else build(t, q, q_next, q)
            Kn = _cmm(_cmm(U, K) * m.mk, U.conj().T) * m.mk
            Kh = Kn.conj().T
            herm = float((Kn - Kh).norm() / Kn.norm())
            K_new = 0.5 * (Kn + Kh)
            q_next = m.charges(K_new)
        K = K_new
        q_prev, q = q, q_next
        unit = math.nan
        if case["unit_every"] and (s + 1) % case["unit_every"] == 0:
            V = m.p(torch.complex(m.S @ U.real.contiguous(), m.S @ U.imag.contiguous()))
            unit = float((m.p(_cmm(U.conj().T, V)) - m.S).norm() / m.S.norm())
        P = -(d * q[:, None]).sum(dim=0)
        rows.append([t + dt, *P.tolist(), float(q.sum()), herm, unit])
    return np.array(rows), K


def _seconds(n, products):
    return 2.0 * float(n) ** 3 * products / 2e13


def exact(case, seed):
    if case["kind"] == "mlp":
        desc, target, w = _mlp_inputs(case, seed)
        b = case["b"]
        n_in, n_out = 4 + b * b, b * b
        W1 = w[:HIDDEN * n_in].astype(np.float16).astype(np.float64).reshape(HIDDEN, n_in)
        o = HIDDEN * n_in
        b1 = w[o:o + HIDDEN].astype(np.float64)
        o += HIDDEN
        W2 = w[o:o + n_out * HIDDEN].astype(np.float16).astype(np.float64).reshape(n_out, HIDDEN)
        b2 = w[o + n_out * HIDDEN:].astype(np.float64)
        x, t = desc.astype(np.float64), target.astype(np.float64)
        h = np.tanh(x @ W1.T + b1)
        y = h @ W2.T + b2
        e = y - t
        dy = 2.0 * e / e.size
        dh = (dy @ W2) * (1.0 - h * h)
        grad = np.concatenate([(dh.T @ x).ravel(), dh.sum(0), (dy.T @ h).ravel(), dy.sum(0)])
        return {"y": y, "loss": float((e * e).mean()), "grad": grad}
    if case["kind"] == "batch":
        res = {}
        for b, xyz, ptr in _batch_members(case):
            if _seconds(len(xyz) * b, 8 + 24 * case["steps"]) > 15.0:
                return None
            x = torch.from_numpy(xyz).to(DEV)
            m = _Dense(x, b, 8.0, 12.0, seed + b)
            X, _ = m.inverse()
            U = m.taylor(m.p(X @ m.H0), case["dt"])
            for k, kappa in enumerate(KICKS):
                K = m.kick(kappa)
                rows = []
                for _ in range(case["steps"]):
                    Kn = _cmm(_cmm(U, K) * m.mk, U.conj().T) * m.mk
                    K = 0.5 * (Kn + Kn.conj().T)
                    q = m.charges(K)
                    row = []
                    for g in range(len(ptr) - 1):
                        s = slice(int(ptr[g]), int(ptr[g + 1]))
                        d = x[s] - x[s].mean(dim=0)
                        row.append([*(-(d * q[s, None]).sum(dim=0)).tolist(), float(q[s].sum())])
                    rows.append(row)
                res["trace%d_%d" % (b, k)] = np.array(rows)
                res["K%d_%d" % (b, k)] = m.blocks(K, m.krows, m.kcols)
        return res
    xyz = _positions(case)
    n = len(xyz) * case["b"]
    if case["kind"] == "inverse":
        if n > 16000:
            return None
        m = _Dense(torch.from_numpy(xyz).to(DEV), case["b"], case["r_hs"], case["r_k"], seed)
        X, iters = m.inverse()
        return {"iterations": iters, "X": m.blocks(X, m.prows, m.pcols).to(torch.complex128)}
    per = {"em": 12, "etrs": 24, "m4": 32}[case["propagator"]]
    if n > 16000 or _seconds(n, 12 + per * (case["steps"] + 2 * case["corrector"])) > 15.0:
        return None
    m = _Dense(torch.from_numpy(xyz).to(DEV), case["b"], case["r_hs"], case["r_k"], seed)
    trace, K = _exact_steps(m, case, _kappa(seed))
    return {"trace": trace, "K": m.blocks(K, m.krows, m.kcols)}
