"""The work that users of the library have it do, as cases to measure.

Every case calls a public entry point of `paper_2503_16717_amd.binding` the way a program does: one library
context for the process, device-resident blocks or matrices, results in the caller's buffers.

kinds of cases
  block    one BCGS2 block step [Q_j, R_j] = qr(Q, V): what an s-step solver of the caller's own runs per
           s vectors (`orth_block`, or the entry point that allocates nothing)
  blocks   the block QR of a whole tall matrix of nb blocks (`orth_blocks`), one-stage or two-stage,
           FP64 or FP32 storage
  sketch   Theta^T X of a tall block (`sketch_apply`)
  gmres    s-step GMRES on a stencil matrix with a fixed budget of basis vectors, as the inner solve of an
           outer iteration has it (the tolerance is not reached within the budget)
  batch    many independent 2-D solves of uneven size advanced together, with a fixed budget

Inputs.  Blocks are n x w with singular values log-spaced from 1 to 10^-e on random orthonormal factors (tall
Gaussian matrices, whose columns are orthonormal up to 1/sqrt(n)), plus a random combination of the block before
them, as successive Krylov panels lean on each other.  Matrices are the integer Laplacian stencils and the
upwind convection-diffusion stencils of the repository's workloads, with the winds and right-hand sides drawn.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2503_16717_amd import binding as B

DEV = "cuda"
_CTX = {}


def _context():
    """The process's library context (one handle, kept, as a program keeps it)."""
    if "ctx" not in _CTX:
        _CTX["ctx"] = B.Context(0)
    return _CTX["ctx"]


# --------------------------------------------------------------------------------------
# the cases
# --------------------------------------------------------------------------------------
def listed():
    return [
        # one s = 5 block step of the 100 x 100 Laplacian in the middle of a restart cycle, Gaussian
        # sketch of 24 rows, through the entry point for loops that may not allocate: pure latency
        dict(name="block_n1e4_w6", kind="block", n=10_000, p=25, w=6, mixed=False, noalloc=True,
             intra="randcholqr", sketch="gaussian", k=24, zeta=0, e=4.0),
        # an s = 10 block step on an odd number of rows (no column but the first is aligned)
        dict(name="block_n1e6_w11_odd", kind="block", n=1_000_003, p=40, w=11, mixed=False, noalloc=False,
             intra="randcholqr", sketch="sparse_sign", k=64, zeta=8, e=4.0),
        # the same step with FP32 storage, four million rows
        dict(name="block_mixed_n4e6_w11", kind="block", n=4_000_037, p=50, w=11, mixed=True, noalloc=False,
             intra="randcholqr", sketch="sparse_sign", k=64, zeta=8, e=1.0),
        # block QR of a small problem by CholQR2-BCGS2, the scheme without a sketch
        dict(name="blocks_cholqr2_n3e5", kind="blocks", n=300_000, nb=8, w=5, two_stage=False, ppb=1,
             mixed=False, intra="cholqr2", preproc="randbcgs2", sketch="sparse_sign", k=64, zeta=8, e=4.0),
        # the repository's headline workload: 12 blocks of 6 columns, 2^24 rows, sparse-sign sketch
        dict(name="blocks_1stage_n2p24", kind="blocks", n=1 << 24, nb=12, w=6, two_stage=False, ppb=1,
             mixed=False, intra="randcholqr", preproc="randbcgs2", sketch="sparse_sign", k=64, zeta=8, e=4.0),
        # the same matrix by the two-stage scheme, big panels of 36 columns
        dict(name="blocks_2stage_n2p24", kind="blocks", n=1 << 24, nb=12, w=6, two_stage=True, ppb=6,
             mixed=False, intra="randcholqr", preproc="randbcgs2", sketch="sparse_sign", k=64, zeta=8, e=4.0),
        # FP32 storage at s = 10: 12 blocks of 11 columns
        dict(name="blocks_mixed_n2p24", kind="blocks", n=1 << 24, nb=12, w=11, two_stage=False, ppb=1,
             mixed=True, intra="randcholqr", preproc="randbcgs2", sketch="sparse_sign", k=64, zeta=8, e=1.0),
        # two-stage QR of an odd-sized matrix with the sketch-free BCGS-PIP pre-processing
        dict(name="blocks_pip_n1e6_odd", kind="blocks", n=1_048_573, nb=8, w=6, two_stage=True, ppb=4,
             mixed=False, intra="randcholqr", preproc="pip", sketch="sparse_sign", k=64, zeta=8, e=3.0),
        # the 128-row sketch of an s = 10 panel of the 192^3 problem
        dict(name="sketch_n7e6_w11", kind="sketch", n=192 ** 3, w=11, mixed=False, sketch="sparse_sign", k=128,
             zeta=8),
        # the 100 x 100 Laplacian, s = 5, restart 30: launch latency and small steps
        dict(name="gmres_laplace2d_100", kind="gmres", dim=2, N=100, wind=False, s=5, m=30, shat=0,
             two_stage=False, jacobi=False, mixed=False, sketch="gaussian", k=24, zeta=0, budget=300),
        # 3-D convection-diffusion on 192^3, Jacobi, two-stage with one big panel per cycle
        dict(name="gmres_convdiff3d_192", kind="gmres", dim=3, N=192, wind=True, s=5, m=60, shat=60,
             two_stage=True, jacobi=True, mixed=False, sketch="sparse_sign", k=128, zeta=8, budget=120),
        # 64 independent 2-D convection-diffusion systems of uneven size, in lock step
        dict(name="batch_convdiff2d_64", kind="batch", nsys=64, lo=64, hi=512, s=5, m=40, shat=20, jacobi=True,
             mixed=False, k=48, zeta=8, budget=80),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["block", "block", "blocks", "blocks", "blocks", "sketch", "gmres", "gmres", "batch"])
    if kind == "block":
        w = rng.choice([4, 5, 6, 6, 8, 11, 11, 13, 16])
        sk = rng.choice(["gaussian", "sparse_sign", "sparse_sign"])
        n = _logint(rng, 4_000, 1 << 23)
        if rng.random() < 0.5:
            n |= 1
        mixed = rng.random() < 0.3
        k = 32 if sk == "gaussian" else rng.choice([48, 64, 128])
        return dict(kind=kind, n=n, p=rng.randint(0, 5) * (w - 1) if rng.random() < 0.7 else rng.randint(1, 72),
                    w=w, mixed=mixed, noalloc=rng.random() < 0.3 and k * w <= 1536,  # its fixed scratch
                    intra=rng.choice(["randcholqr", "cholqr2"]), sketch=sk, k=k,
                    zeta=0 if sk == "gaussian" else rng.choice([4, 8]), e=1.0 if mixed else rng.choice([2.0, 4.0]))
    if kind == "blocks":
        w = rng.choice([4, 5, 6, 6, 8, 11, 12])
        nb = rng.choice([4, 6, 8, 12])
        two = rng.random() < 0.5
        ppb = rng.choice([q for q in (2, 3, 4, 6) if nb % q == 0 and q * w <= 64]) if two else 1
        mixed = rng.random() < 0.3
        n = _logint(rng, 20_000, min(1 << 24, (72 << 24) // (nb * w) * 2 // 3))
        if rng.random() < 0.4:
            n |= 1
        return dict(kind=kind, n=n, nb=nb, w=w, two_stage=two, ppb=ppb, mixed=mixed,
                    intra=rng.choice(["randcholqr", "randcholqr", "cholqr2"]),
                    preproc="pip" if two and not mixed and rng.random() < 0.25 else "randbcgs2",
                    sketch="sparse_sign", k=128 if ppb * w > 40 else rng.choice([64, 128]), zeta=8,
                    e=1.0 if mixed else rng.choice([2.0, 3.0]))
    if kind == "sketch":
        n = _logint(rng, 10_000, 1 << 24)
        if rng.random() < 0.5:
            n |= 1
        return dict(kind=kind, n=n, w=rng.choice([4, 6, 6, 9, 11, 11, 16]), mixed=rng.random() < 0.3,
                    sketch="sparse_sign", k=rng.choice([48, 64, 96, 128, 256]), zeta=rng.choice([2, 4, 8, 8]))
    if kind == "gmres":
        dim = rng.choice([2, 3])
        s = rng.choice([4, 5, 5, 6])
        two = rng.random() < 0.6
        cyc = rng.choice([3, 4, 6])
        m = s * cyc
        shat = s * rng.choice([q for q in range(1, cyc + 1) if cyc % q == 0]) if two else 0
        N = _logint(rng, 64, 1200) if dim == 2 else _logint(rng, 20, 160)
        gauss = N ** dim < 300_000 and rng.random() < 0.3
        return dict(kind=kind, dim=dim, N=N, wind=rng.random() < 0.6, s=s, m=m, shat=shat, two_stage=two,
                    jacobi=rng.random() < 0.5, mixed=False, sketch="gaussian" if gauss else "sparse_sign",
                    k=64 if gauss else 128, zeta=0 if gauss else 8, budget=2 * m)
    lo = rng.choice([32, 48, 64])
    return dict(kind="batch", nsys=rng.randint(8, 64), lo=lo, hi=lo * rng.choice([2, 4, 6]), s=5, m=40, shat=20,
                jacobi=rng.random() < 0.6, mixed=False, k=48, zeta=8, budget=40)


# --------------------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------------------
def _generator(seed, salt):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1_000_003 + salt * 7919) & 0x7FFF_FFFF_FFFF)
    return g


def _columns(n, N, dtype):
    """An uninitialised column-major n x N tensor."""
    return torch.empty((N, n), dtype=dtype, device=DEV).t()


def _rotation(w, g):
    return torch.linalg.qr(torch.randn((w, w), dtype=torch.float64, device=DEV, generator=g).cpu())[0].to(DEV)


def _fill_block(out, e, g, lean=None):
    """out (n x w column-major view) = G diag(sigma) W^T (+ lean @ M)."""
    n, w = out.shape
    sigma = 10.0 ** (-e * torch.arange(w, dtype=torch.float64, device=DEV) / max(1, w - 1))
    mix = sigma[:, None] * _rotation(w, g).t() / math.sqrt(n)
    lm = None
    if lean is not None:
        lm = 0.3 * torch.randn((lean.shape[1], w), dtype=torch.float64, device=DEV, generator=g) / math.sqrt(w)
    step = 1 << 22
    for r in range(0, n, step):
        c = min(step, n - r)
        blk = mix.t() @ torch.randn((w, c), dtype=torch.float64, device=DEV, generator=g)
        if lean is not None:
            blk += lm.t() @ lean[r:r + c].t().double()
        out[r:r + c].copy_(blk.t())


def _theta_gaussian(n, k, g):
    return (torch.randn((k, n), dtype=torch.float64, device=DEV, generator=g) / math.sqrt(k)).t()


def _sketch(case, seed, n, g):
    if case["sketch"] == "gaussian":
        th = _theta_gaussian(n, case["k"], g)
        return B.make_sketch("gaussian", theta=th), th
    return B.make_sketch("sparse_sign", case["k"], case["zeta"], int(seed) & 0xFFFF), None


def _stencil(dim, N, wind):
    """(centre, lower, upper) of the stencil: unscaled Laplacian, or upwind convection-diffusion times h^2."""
    if wind is None:
        return 2.0 * dim, [-1.0] * dim, [-1.0] * dim
    h = 1.0 / (N + 1)
    return 2.0 * dim + h * sum(wind), [-1.0 - h * b for b in wind], [-1.0] * dim


def _csr(dim, N, wind):
    """CSR tensors (int32 row pointers and sorted column indices, float64 values) on the device."""
    centre, lower, upper = _stencil(dim, N, wind)
    n = N ** dim
    i = torch.arange(n, dtype=torch.int64, device=DEV)
    cols, vals, ok = [], [], []
    for d, o in [(d, -1) for d in reversed(range(dim))] + [(0, 0)] + [(d, 1) for d in range(dim)]:
        x = (i // N ** d) % N
        cols.append(i + o * N ** d)
        vals.append(centre if o == 0 else (lower[d] if o < 0 else upper[d]))
        ok.append((x + o >= 0) & (x + o < N))
    ok = torch.stack(ok, 1)
    rowptr = torch.zeros(n + 1, dtype=torch.int32, device=DEV)
    rowptr[1:] = torch.cumsum(ok.sum(1), 0).to(torch.int32)
    colind = torch.stack(cols, 1)[ok].to(torch.int32)
    val = torch.tensor(vals, dtype=torch.float64, device=DEV).expand(n, -1)[ok]
    return rowptr, colind, val


def _sko_csr(rowptr, colind, val):
    s = B.sko_csr()
    s.n, s.nnz = rowptr.shape[0] - 1, val.shape[0]
    s.rowptr, s.colind, s.val = rowptr.data_ptr(), colind.data_ptr(), val.data_ptr()
    return s


def _winds(case, seed):
    """The wind of a solve (None: Laplacian), or (grid side, wind) of a batch's systems, whose sides
    are spread evenly over the logarithm of the case's range."""
    r = np.random.default_rng([11, int(seed)])
    if case["kind"] == "gmres":
        return [float(v) for v in r.uniform(5.0, 40.0, case["dim"])] if case["wind"] else None
    ns, ratio = case["nsys"], math.log(case["hi"] / case["lo"])
    return [(int(round(case["lo"] * math.exp(ratio * ((7 * i) % ns + 0.5) / ns))),
             [float(v) for v in r.uniform(0.0, 50.0, 2)]) for i in range(ns)]


def _gmres_kw(case, sk):
    return dict(s=case["s"], m=case["m"], shat=case["shat"], two_stage=case.get("two_stage", True),
                precond=1 if case["jacobi"] else 0, precision="mixed" if case["mixed"] else "f64", sketch=sk,
                tol=1e-14, maxiter=case["budget"])


def prepare(case, seed):
    ctx = _context()
    kind = case["kind"]
    g = _generator(seed, 1)
    st = dict(kind=kind, ctx=ctx)
    if kind in ("block", "blocks", "sketch"):
        dt = torch.float32 if case["mixed"] else torch.float64
        n, w = case["n"], case["w"]
        st["sk"], st["keep"] = _sketch(case, seed, n, g)
        st["precision"] = "mixed" if case["mixed"] else "f64"
        if kind == "block":
            p = case["p"]
            st["Q"] = None
            lean = None
            if p > 0:
                Q = torch.randn((p, n), dtype=torch.float64, device=DEV, generator=g)
                for _ in range(2):
                    Q = torch.linalg.inv(torch.linalg.cholesky((Q @ Q.t()).cpu())).to(DEV) @ Q
                st["Q"] = Q.to(dt).contiguous().t()
                lean = st["Q"]
            st["V"] = _columns(n, w, dt)
            _fill_block(st["V"], case["e"], g, lean)
            st["out"] = _columns(n, w, dt)
            st["noalloc"] = case["noalloc"]
            st["opts"] = dict(intra=case["intra"], precision=st["precision"], sketch=st["sk"])
        elif kind == "blocks":
            N = case["nb"] * w
            st["V"] = _columns(n, N, dt)
            for j in range(case["nb"]):
                _fill_block(st["V"][:, j * w:(j + 1) * w], case["e"], g,
                            st["V"][:, (j - 1) * w:j * w] if j else None)
            st["out"] = _columns(n, N, dt)
            st["w"] = w
            st["opts"] = dict(intra=case["intra"], two_stage=case["two_stage"], panels_per_big=case["ppb"],
                              precision=st["precision"], preproc=case["preproc"], sketch=st["sk"])
        else:
            st["V"] = _columns(n, w, dt)
            _fill_block(st["V"], 2.0, g)
        return st
    if kind == "gmres":
        n = case["N"] ** case["dim"]
        st["csr"] = _csr(case["dim"], case["N"], _winds(case, seed))
        st["A"] = _sko_csr(*st["csr"])
        st["sk"], st["keep"] = _sketch(case, seed, n, g)
        st["b"] = torch.rand(n, dtype=torch.float64, device=DEV, generator=g) * 2.0 - 1.0
        st["kw"] = _gmres_kw(case, st["sk"])
        return st
    sizes = _winds(case, seed)
    st["csr"] = [_csr(2, N, wind) for N, wind in sizes]
    st["A"] = [_sko_csr(*c) for c in st["csr"]]
    ns = [N * N for N, _ in sizes]
    offs = [0]
    for v in ns:
        offs.append(offs[-1] + (v + 63) // 64 * 64)
    st["spans"] = [(o, o + v) for o, v in zip(offs, ns)]
    st["b"] = torch.rand(offs[-1], dtype=torch.float64, device=DEV, generator=g) * 2.0 - 1.0
    st["x"] = torch.zeros(offs[-1], dtype=torch.float64, device=DEV)
    st["bp"] = [st["b"].data_ptr() + 8 * o for o in offs[:-1]]
    st["xp"] = [st["x"].data_ptr() + 8 * o for o in offs[:-1]]
    st["opts"] = B.gmres_opts(**_gmres_kw(case, B.make_sketch("sparse_sign", case["k"], case["zeta"],
                                                              int(seed) & 0xFFFF)))
    return st


# --------------------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------------------
def run(st):
    ctx, kind = st["ctx"], st["kind"]
    if kind == "block":
        Q, Rp, Rd, status, _ = ctx.orth_block(st["Q"], st["V"], st["out"], noalloc=st["noalloc"], **st["opts"])
        return {"Q": Q, "R_proj": Rp, "R_diag": Rd, "status": int(status)}
    if kind == "blocks":
        Q, R, status, _ = ctx.orth_blocks(st["V"], st["w"], Q=st["out"], **st["opts"])
        return {"Q": Q, "R": R, "status": int(status)}
    if kind == "sketch":
        return {"Y": ctx.sketch_apply(st["V"], st["sk"], st["precision"])}
    if kind == "gmres":
        x, info, status = ctx.gmres((st["A"], st["csr"]), st["b"], **st["kw"])
        return {"x": x, "iters": int(info["iters"]), "status": int(status)}
    st["x"].zero_()
    status, infos = ctx.sko_gmres_batched(st["A"], st["bp"], st["xp"], st["opts"])
    return {"x": st["x"], "iters": [int(sum(i.iters for i in infos))], "status": int(status)}


# --------------------------------------------------------------------------------------
# the bytes and operations a pass cannot do without
# --------------------------------------------------------------------------------------
def work(case):
    kind = case["kind"]
    if kind in ("block", "blocks", "sketch"):
        eb = 4 if case["mixed"] else 8
        n, w = case["n"], case["w"]
        if kind == "sketch":
            return {"bytes": n * w * eb, "flops": 2 * n * w * case["zeta"]}
        if kind == "block":
            p = case["p"]
            return {"bytes": n * (p + 2 * w) * eb + (8 * n * case["k"] if case["zeta"] == 0 and
                                                     case["intra"] == "randcholqr" else 0),
                    "flops": n * w * (8 * p + 4 * w)}
        N = case["nb"] * w
        return {"bytes": 2 * n * N * eb, "flops": 4 * n * N * N}
    if kind == "gmres":
        n = case["N"] ** case["dim"]
        per = 2 * case["dim"] + 1
        nnz = per * n - 2 * case["dim"] * case["N"] ** (case["dim"] - 1)
        vec, m, ns, nn = (4 if case["mixed"] else 8), case["m"], case["budget"], float(n)
    else:
        side2 = (case["hi"] ** 2 - case["lo"] ** 2) / (2 * math.log(case["hi"] / case["lo"]))
        nn = case["nsys"] * side2
        nnz = 5 * nn
        vec, m, ns = (4 if case["mixed"] else 8), case["m"], case["budget"]
    # per basis vector: the operator once, its input and output vector once; per cycle the basis once more to
    # orthogonalise it (read and written) and once for the solution
    return {"bytes": ns * (nnz * (vec + 4) + nn * (4 + 2 * vec)) + ns * nn * 3 * vec,
            "flops": ns * (2 * nnz + nn * 4 * m)}


# --------------------------------------------------------------------------------------
# the same results in 64 bits with plain torch
# --------------------------------------------------------------------------------------
def _gram(X, Y):
    """X^T Y of tall row-chunked operands (n x a, n x b), summed over chunks in FP64."""
    s = torch.zeros((X.shape[1], Y.shape[1]), dtype=torch.float64, device=DEV)
    for r in range(0, X.shape[0], 1 << 20):
        s += X[r:r + (1 << 20)].t() @ Y[r:r + (1 << 20)]
    return s


def _apply_inv(X, R):
    """X R^{-1} in place, in row chunks."""
    Rt = R.t().contiguous()
    for r in range(0, X.shape[0], 1 << 18):
        c = X[r:r + (1 << 18)]
        c.copy_(torch.linalg.solve_triangular(Rt, c.t().contiguous(), upper=False).t())


def _exact_block(Q, V):
    """Block Gram-Schmidt with Cholesky QR, three passes: (Q_j, R_proj, R_diag)."""
    w = V.shape[1]
    X = V.double().t().contiguous().t()
    Rp = None if Q is None else torch.zeros((Q.shape[1], w), dtype=torch.float64, device=DEV)
    Rd = torch.eye(w, dtype=torch.float64, device=DEV)
    for _ in range(3):
        if Q is not None:
            C = _gram(Q, X)
            for r in range(0, X.shape[0], 1 << 20):
                X[r:r + (1 << 20)] -= Q[r:r + (1 << 20)] @ C
            Rp += C @ Rd
        R = torch.linalg.cholesky(_gram(X, X)).t()
        _apply_inv(X, R)
        Rd = R @ Rd
    return X, Rp, Rd


def _splitmix(seed, n):
    """SplitMix64 output i + 1 of the stream started at `seed`, i = 0..n-1, as int64 bits."""
    def sx(v):
        return v - (1 << 64) if v >= 1 << 63 else v

    def shr(z, k):
        return (z >> k) & ((1 << (64 - k)) - 1)

    z = torch.arange(1, n + 1, dtype=torch.int64, device=DEV) * sx(0x9E3779B97F4A7C15) + sx(seed)
    z = (z ^ shr(z, 30)) * sx(0xBF58476D1CE4E5B9)
    z = (z ^ shr(z, 27)) * sx(0x94D049BB133111EB)
    return z ^ shr(z, 31)


def _exact_sketch(case, seed, V):
    n, w = V.shape
    k, zeta = case["k"], case["zeta"]
    Bk = k // zeta
    h = _splitmix(int(seed) & 0xFFFF, n)
    Y = torch.zeros((k, w), dtype=torch.float64, device=DEV)
    for t in range(zeta):
        b = (h >> (8 * t)) & 0xFF
        slot = t * Bk + (((b >> 1) * Bk) >> 7)
        sign = 1.0 - 2.0 * (b & 1).double()
        for j in range(Bk):
            at = (slot == t * Bk + j).nonzero().flatten()
            Y[t * Bk + j] = (V[at].double() * sign[at, None]).sum(0)
    return Y / math.sqrt(zeta)


def _exact_gmres(dim, N, wind, jacobi, m, budget, b):
    """Restarted GMRES(m) with right Jacobi, `budget` Krylov vectors in all, from x0 = 0."""
    centre, lower, upper = _stencil(dim, N, wind)
    shape = (N,) * dim

    def A(v):
        v = v.view(shape)
        y = centre * v
        for d in range(dim):
            ax = dim - 1 - d
            y.narrow(ax, 1, N - 1).add_(v.narrow(ax, 0, N - 1), alpha=lower[d])
            y.narrow(ax, 0, N - 1).add_(v.narrow(ax, 1, N - 1), alpha=upper[d])
        return y.reshape(-1)

    dinv = 1.0 / centre if jacobi else 1.0
    x = torch.zeros_like(b)
    done = 0
    while done < budget:
        r = b - A(x)
        beta = r.norm()
        V = torch.empty((m + 1, b.shape[0]), dtype=torch.float64, device=DEV)
        V[0] = r / beta
        H = torch.zeros((m + 1, m), dtype=torch.float64, device=DEV)
        for j in range(m):
            u = A(V[j]) * dinv
            for _ in range(2):
                c = V[:j + 1] @ u
                u = u - c @ V[:j + 1]
                H[:j + 1, j] += c
            H[j + 1, j] = u.norm()
            V[j + 1] = u / H[j + 1, j]
        rhs = torch.zeros(m + 1, dtype=torch.float64)
        rhs[0] = beta.item()
        y = torch.linalg.lstsq(H.cpu(), rhs[:, None]).solution[:, 0].to(DEV)
        x = x + dinv * (y @ V[:m])
        done += m
    return x


def exact(case, seed):
    kind = case["kind"]
    st = prepare(case, seed)
    if kind == "block":
        Q, Rp, Rd = _exact_block(None if st["Q"] is None else st["Q"].double(), st["V"])
        return {"Q": Q, "R_proj": Rp, "R_diag": Rd, "status": None}
    if kind == "blocks":
        V, w, nb = st["V"], case["w"], case["nb"]
        n, N = V.shape
        Q = torch.empty((N, n), dtype=torch.float64, device=DEV).t()
        R = torch.zeros((N, N), dtype=torch.float64, device=DEV)
        for j in range(nb):
            p = j * w
            Qj, Rp, Rd = _exact_block(Q[:, :p] if p else None, V[:, p:p + w])
            Q[:, p:p + w] = Qj
            R[p:p + w, p:p + w] = Rd
            if p:
                R[:p, p:p + w] = Rp
        return {"Q": Q, "R": R, "status": None}
    if kind == "sketch":
        return {"Y": _exact_sketch(case, seed, st["V"])}
    if kind == "gmres":
        x = _exact_gmres(case["dim"], case["N"], _winds(case, seed), case["jacobi"], case["m"], case["budget"],
                         st["b"])
        return {"x": x, "iters": None, "status": None}
    x = torch.zeros_like(st["x"])
    for (lo, hi), (N, wind) in zip(st["spans"], _winds(case, seed)):
        x[lo:hi] = _exact_gmres(2, N, wind, case["jacobi"], case["m"], case["budget"], st["b"][lo:hi])
    return {"x": x, "iters": None, "status": None}
