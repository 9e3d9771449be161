"""The matrix-powers operator by diagonals or as CSR: matrices on either side of each condition of
the choice (number of diagonals, padding, column order) must solve alike.  Tolerances: the
explicit relative residual at the solver's tolerance, and x within the tolerance times the
condition number of the diagonally dominant test matrices (at most 100) of a direct solve."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2503_16717_amd import workloads as wl  # noqa: E402

pytestmark = pytest.mark.gpu
TOL = 1e-11


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_16717_amd import binding
    return binding


@pytest.fixture(scope="module")
def ctx(B):
    c = B.Context(0)
    yield c
    c.close()


def banded(n, offsets, seed, drop=0.0):
    """Diagonally dominant matrix with random values on the given diagonals (a share dropped)."""
    r = np.random.default_rng([21, seed])
    rows, cols, vals = [], [], []
    i = np.arange(n)
    for o in offsets:
        ok = (i + o >= 0) & (i + o < n) & ((r.uniform(size=n) >= drop) | (o == 0))
        rows.append(i[ok])
        cols.append(i[ok] + o)
        v = r.uniform(-1.0, 1.0, ok.sum()) if o else np.full(ok.sum(), 1.5 * len(offsets))
        vals.append(v)
    rows, cols, vals = map(np.concatenate, (rows, cols, vals))
    order = np.lexsort((cols, rows))
    rowptr = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(np.bincount(rows, minlength=n), out=rowptr[1:])
    return wl.CSR(n, rowptr, cols[order], vals[order])


def csr_twin(A):
    """The same matrix with one row's entries out of order, which keeps it off the diagonal form."""
    row = int(np.argmax(np.diff(A.rowptr) > 1))
    e0, e1 = A.rowptr[row], A.rowptr[row + 1]
    T = wl.CSR(A.n, A.rowptr.copy(), A.colind.copy(), A.val.copy())
    T.colind[e0:e1] = T.colind[e0:e1][::-1].copy()
    T.val[e0:e1] = T.val[e0:e1][::-1].copy()
    return T


def solve_and_check(B, ctx, A, **kw):
    import scipy.sparse.linalg as sla
    b = wl.rhs_uniform(A.n, 3)
    x, info, st = ctx.gmres(A, b, tol=TOL, **kw)
    if st != B.SKO_OK:
        # nearly a multiple of the identity: the Krylov space is exhausted, in either form
        assert st == B.SKO_EBREAKDOWN and ctx.gmres(csr_twin(A), b, tol=TOL, **kw)[2] == st, (st, info)
        return
    S = A.to_scipy().tocsc()
    x = x.cpu().numpy()
    assert np.linalg.norm(b - S @ x) / np.linalg.norm(b) <= TOL
    ref = sla.spsolve(S, b)
    assert np.linalg.norm(x - ref) <= 100 * TOL * np.linalg.norm(ref)


CASES = {
    "1 diagonal": (700, [0], 0.0),
    "3 diagonals": (513, [-1, 0, 1], 0.0),
    "upper only": (1000, [0, 1, 7, 300], 0.0),
    "far corners": (600, [-599, 0, 599], 0.0),
    "16 diagonals": (2049, sorted([-900, -400, -77, -30, -9, -3, -2, -1, 0, 1, 2, 5, 11, 64, 500, 1000]), 0.0),
    "17 diagonals": (2049, sorted([-901, -900, -400, -77, -30, -9, -3, -2, -1, 0, 1, 2, 5, 11, 64, 500, 1000]), 0.0),
    "part-filled": (3000, [-40, -5, -1, 0, 1, 5, 40], 0.7),
    "a few gaps": (3000, [-40, -1, 0, 1, 40], 0.05),
}


@pytest.mark.parametrize("name", CASES)
@pytest.mark.parametrize("precision", ["f64", "mixed"])
def test_diagonal_counts(B, ctx, name, precision):
    n, offs, drop = CASES[name]
    A = banded(n, offs, len(name), drop)
    sk = B.make_sketch("sparse_sign", 64, 8, 1)
    for kw in (dict(s=4, m=12), dict(s=4, m=12, two_stage=True, shat=12, precond=1)):
        if len(offs) == 1 and kw.get("precond"):
            # A D^{-1} = I: every Krylov vector equals the first (which column of rounding noise gives
            # the first non-positive pivot depends on the storage)
            assert ctx.gmres(A, wl.rhs_uniform(n, 3), tol=TOL, precision=precision, sketch=sk,
                             **kw)[2] == B.SKO_EBREAKDOWN
            continue
        solve_and_check(B, ctx, A, precision=precision, sketch=sk, **kw)


def test_rows_out_of_order_keep_csr(B, ctx):
    A = csr_twin(banded(900, [-3, 0, 3], 5))
    solve_and_check(B, ctx, A, s=4, m=12, sketch=B.make_sketch("sparse_sign", 64, 8, 1))


@pytest.mark.parametrize("basis", ["monomial", "newton"])
def test_two_rows_per_thread(B, ctx, basis):
    """Above the size at which a thread takes two rows, odd row count."""
    A = banded((1 << 18) + 261, [-513, -1, 0, 1, 513], 8)
    solve_and_check(B, ctx, A, s=4, m=12, basis=basis, sketch=B.make_sketch("sparse_sign", 64, 8, 1))


def test_batch_of_mixed_forms(B, ctx):
    """One system of a batch off the diagonal form: the whole batch runs on CSR."""
    for offs in ([-2, 0, 2], list(range(-9, 10))):
        systems = [banded(400 + 37 * i, [-20, -1, 0, 1, 20], i) for i in range(3)] + [banded(777, offs, 9)]
        dev = [B.csr_to_device(A) for A in systems]
        bs = [torch.from_numpy(wl.rhs_uniform(A.n, 3)).cuda() for A in systems]
        xs = [torch.zeros_like(b) for b in bs]
        o = B.gmres_opts(s=4, m=12, shat=12, two_stage=True, precond=1, tol=TOL,
                         sketch=B.make_sketch("sparse_sign", 64, 8, 1))
        st, infos = ctx.sko_gmres_batched([d[0] for d in dev], [b.data_ptr() for b in bs], [x.data_ptr() for x in xs], o)
        assert st == B.SKO_OK
        for A, b, x in zip(systems, bs, xs):
            b, x = b.cpu().numpy(), x.cpu().numpy()
            assert np.linalg.norm(b - A.to_scipy() @ x) / np.linalg.norm(b) <= TOL


def coupled_fields(N, dim=2):
    """Two stencil fields that share a unit coupling: diagonals at both ends of the matrix, so no
    stretch of rows has every diagonal inside it."""
    import scipy.sparse as sp
    S = (wl.convdiff_2d(N, 10.0, 20.0) if dim == 2 else wl.convdiff_3d(N, (5.0, 10.0, 15.0))).to_scipy()
    S = S + sp.identity(S.shape[0])
    T = sp.bmat([[S, 0.1 * sp.identity(S.shape[0])], [-0.1 * sp.identity(S.shape[0]), S]]).tocsr()
    T.sort_indices()
    return wl.CSR(T.shape[0], T.indptr.astype(np.int64), T.indices, T.data)


def spmv_kernels(ctx, solve, repeats=5):
    """{kernel name: mean microseconds} of the matrix-powers launches of `solve`, the best of several runs."""
    best = {}
    for _ in range(repeats):
        ctx.sko_profile_enable(True)
        solve()
        for k in ctx.sko_profile_read():
            if k["name"].startswith("spmv"):
                t = 1e3 * k["total_ms"] / k["launches"]
                best[k["name"]] = min(t, best.get(k["name"], t))
        ctx.sko_profile_enable(False)
    return best


# 2 x 12^2 rows: one workgroup; 2 x 31^2: a ragged last one; 2 x 400^2: two rows per thread
@pytest.mark.parametrize("N,dim", [(12, 2), (31, 2), (400, 2), (9, 3)])
@pytest.mark.parametrize("precision", ["f64", "mixed"])
def test_coupled_fields_solve(B, ctx, N, dim, precision):
    A = coupled_fields(N, dim)
    b = wl.rhs_uniform(A.n, 3)
    kw = dict(s=4, m=12, precond=1, precision=precision, tol=1e-8, maxiter=4000,
              sketch=B.make_sketch("sparse_sign", 64, 8, 1))
    assert list(spmv_kernels(ctx, lambda: ctx.gmres(A, b, **kw), 1)) == [
        "spmv dia " + ("f32" if precision == "mixed" else "f64")]
    for two in (dict(), dict(two_stage=True, shat=12)):
        x, info, st = ctx.gmres(A, b, **kw, **two)
        assert st == B.SKO_OK, (st, info)
        assert np.linalg.norm(b - A.to_scipy() @ x.cpu().numpy()) / np.linalg.norm(b) <= 1e-8


@pytest.mark.parametrize("precision", ["f64", "mixed"])
def test_coupled_fields_are_no_slower_by_diagonals(B, ctx, precision):
    """The form is chosen for its fewer bytes; every workgroup of this matrix has a diagonal outside."""
    A = coupled_fields(1000)
    b = wl.rhs_uniform(A.n, 3)
    kw = dict(s=5, m=20, precision=precision, tol=1e-14, maxiter=20, sketch=B.make_sketch("sparse_sign", 64, 8, 1))
    dia = spmv_kernels(ctx, lambda: ctx.gmres(A, b, **kw))
    csr = spmv_kernels(ctx, lambda: ctx.gmres(csr_twin(A), b, **kw))
    print(dia, csr, flush=True)
    ty = "f32" if precision == "mixed" else "f64"
    assert list(dia) == [f"spmv dia {ty}"] and list(csr) == [f"spmv {ty}"]
    assert dia[f"spmv dia {ty}"] <= csr[f"spmv {ty}"]


def with_values(n, offsets, seed, extra=()):
    """A matrix on the given diagonals with a varying dominant main diagonal, and single entries
    (row, column, value) besides."""
    import scipy.sparse as sp
    r = np.random.default_rng([22, seed])
    S = sp.lil_matrix((n, n))
    for o in offsets:
        S.setdiag(r.uniform(-1.0, 1.0, n) if o else len(offsets) * r.uniform(0.7, 1.4, n), o)
    for i, j, v in extra:
        S[i, j] = v
    S = S.tocsr()
    S.sort_indices()
    return wl.CSR(n, S.indptr.astype(np.int64), S.indices, S.data)


BAND5, BAND13 = [-30, -1, 0, 1, 30], list(range(-6, 7))
# name: (matrix, by diagonals)
STRUCTURES = {
    "one row": (lambda: with_values(1, [0], 1), True),
    "fewer rows than samples": (lambda: with_values(40, [-1, 0, 1], 2), True),
    "a whole row block": (lambda: with_values(256, BAND5, 3), True),
    "one row more": (lambda: with_values(257, BAND5, 4), True),
    "rows in two parts": (lambda: with_values(1500, BAND13, 5), True),
    "a diagonal of one entry": (lambda: with_values(3000, BAND5, 6, [(1777, 200, 0.5)]), True),
    "a 17th diagonal of one entry": (
        lambda: with_values(3000, list(range(-8, 8)), 7, [(1777, 200, 0.5)]), False),
    "a row of 17 entries": (
        lambda: with_values(3000, BAND5, 8, [(1501, 1000 + 7 * i, 0.05) for i in range(12)]), False),
    "random columns": (
        lambda: with_values(900, [0], 9, [(i, (i * 37 + 11 * j * j) % 900, 0.1) for i in range(900) for j in range(1, 5)]),
        False),
}


@pytest.mark.parametrize("name", STRUCTURES)
@pytest.mark.parametrize("precond", [0, 1])
def test_structure_scan(B, ctx, name, precond):
    """The scan's shortcuts (sampled rows, rows along the known diagonals) find every diagonal."""
    make, by_diagonals = STRUCTURES[name]
    A = make()
    b = wl.rhs_uniform(A.n, 3)
    kw = dict(s=1 if A.n == 1 else 4, m=1 if A.n == 1 else 12, precond=precond, tol=1e-9,
              maxiter=4 if A.n == 1 else 600, sketch=B.make_sketch("sparse_sign", 64, 8, 1))
    names = list(spmv_kernels(ctx, lambda: ctx.gmres(A, b, **kw), 1))
    assert names == ["spmv dia f64" if by_diagonals else "spmv f64"]
    x, info, st = ctx.gmres(A, b, **kw)
    if A.n > 1:  # a Krylov space of one vector has no second one to orthogonalise
        assert st == B.SKO_OK, (st, info)
        assert np.linalg.norm(b - A.to_scipy() @ x.cpu().numpy()) / np.linalg.norm(b) <= 1e-9


@pytest.mark.parametrize("name", STRUCTURES)
def test_structure_check_rejects(B, ctx, name):
    """One wrong column or row pointer anywhere, in each route of the check."""
    A = STRUCTURES[name][0]()
    b = torch.from_numpy(wl.rhs_uniform(A.n, 3)).cuda()
    kw = dict(s=1, m=1, sketch=B.make_sketch("sparse_sign", 64, 8, 1))

    def status(rowptr, colind, maxiter):
        Ad, keep = B.csr_to_device(A)
        rp, ci = torch.from_numpy(rowptr).cuda(), torch.from_numpy(colind).cuda()
        Ad.rowptr, Ad.colind = rp.data_ptr(), ci.data_ptr()
        return ctx.gmres((Ad, (keep, rp, ci)), b, maxiter=maxiter, **kw)[2]

    for maxiter in (1, 50):  # without and with the scan
        for at in sorted({0, A.nnz // 3, A.nnz // 2, A.nnz - 1}):
            for col in (-1, A.n, 2 ** 31 - 1, -2 ** 31):
                ci = A.colind.copy()
                ci[at] = col
                assert status(A.rowptr, ci, maxiter) == B.SKO_EINVAL, (maxiter, at, col)
        for at in sorted({0, A.n // 2, A.n}):
            for d in (-1, 1, A.nnz + 1, -2 ** 30):
                rp = A.rowptr.copy()
                rp[at] += d
                if rp[0] == 0 and rp[-1] == A.nnz and np.all(np.diff(rp.astype(np.int64)) >= 0):
                    continue  # still a valid structure
                assert status(rp, A.colind, maxiter) == B.SKO_EINVAL, (maxiter, at, d)


def test_short_solves_keep_csr(B, ctx):
    """A solve of fewer vectors than the diagonals' set-up pays for runs as it is."""
    A = wl.laplacian_2d(30)
    b = wl.rhs_uniform(A.n, 3)
    sk = B.make_sketch("sparse_sign", 64, 8, 1)
    for s, maxiter, name in ((3, 3, "spmv f64"), (3, 4, "spmv dia f64"), (4, 1, "spmv dia f64"), (1, 3, "spmv f64")):
        assert list(spmv_kernels(ctx, lambda: ctx.gmres(A, b, s=s, m=4 * s, tol=1e-14, maxiter=maxiter, sketch=sk), 1)) == [name]


BY_DIAGONALS = {"1 diagonal", "3 diagonals", "upper only", "16 diagonals", "a few gaps"}


@pytest.mark.parametrize("name", CASES)
@pytest.mark.parametrize("precision", ["f64", "mixed"])
@pytest.mark.parametrize("scheme", ["one-stage", "two-stage"])
def test_every_form_solves(B, ctx, name, precision, scheme):
    """The structures of CASES with a main diagonal that varies (no early end of the Krylov space): the
    expected form runs, and the residual is checked for every one of them."""
    n, offs, drop = CASES[name]
    A = with_values(n, offs, len(name))
    if drop:
        r = np.random.default_rng([23, len(name)])
        S = A.to_scipy().tocoo()
        keep = (S.row == S.col) | (r.uniform(size=S.nnz) >= drop)
        import scipy.sparse as sp
        S = sp.csr_matrix((S.data[keep], (S.row[keep], S.col[keep])), shape=S.shape)
        S.sort_indices()
        A = wl.CSR(n, S.indptr.astype(np.int64), S.indices, S.data)
    b = wl.rhs_uniform(n, 3)
    kw = dict(s=4, m=12, precision=precision, tol=1e-8, maxiter=2000, sketch=B.make_sketch("sparse_sign", 64, 8, 1))
    if scheme == "two-stage":
        kw.update(two_stage=True, shat=12)
    names = list(spmv_kernels(ctx, lambda: ctx.gmres(A, b, **kw), 1))
    assert len(names) == 1 and names[0].startswith("spmv dia ") == (name in BY_DIAGONALS), names
    x, info, st = ctx.gmres(A, b, **kw)
    assert st == B.SKO_OK, (st, info)
    assert np.linalg.norm(b - A.to_scipy() @ x.cpu().numpy()) / np.linalg.norm(b) <= 1e-8
