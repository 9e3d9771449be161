"""Schedules of whole matrices (sko_orth_blocks): the one-stage look-ahead and the two-stage
sweeps over whole big panels, at the widths, column counts and row remainders where their
kernels change form.  FP64 against the oracle with the bounds of test_gpu_orth.py; FP32 storage
against the sequence of single block steps, which rounds at the same places."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import metrics, orth  # noqa: E402
from oracle.sketch import Sketch  # noqa: E402
from paper_2503_16717_amd import workloads as wl  # noqa: E402

pytestmark = pytest.mark.gpu
U = 2.0 ** -53


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


def tol_r(e):
    return max(1e-12, 10.0 * 10.0 ** e * U)


def check(V, Q, R, ref, e):
    assert ref.info == 0
    assert np.all(np.diag(R) > 0) and np.array_equal(np.tril(R, -1), np.zeros_like(R))
    assert metrics.rel_diff(R, ref.R) <= tol_r(e)
    assert metrics.orth_error(Q)[0] <= 1e-13
    assert metrics.backward_error(V, Q, R) <= 1e-14


# w = 8 | 9: projection tiles of one or two forms, Gram on vector units or MFMA; 12 | 13: the widest
# look-ahead; nb = 2: no middle block; 13 x 11: projections of more than 128 rows in two launches
@pytest.mark.parametrize("w,nb", [(1, 3), (2, 2), (7, 3), (8, 3), (9, 3), (12, 4), (13, 3), (11, 13)])
@pytest.mark.parametrize("n", [255, 4099])
@pytest.mark.parametrize("intra", ["randcholqr", "cholqr2"])
def test_one_stage_edges(B, ctx, w, nb, n, intra):
    if n < nb * w + 32:
        n = 1 + 2 * nb * w
    e = 3.0
    V = wl.glued_blocks(n, nb, w, e)
    Vd = B.colmajor_from_numpy(V, "cuda")
    sk = B.make_sketch("sparse_sign", 64, 8, 5)
    Q, R, st, col = ctx.orth_blocks(Vd, w, intra=intra, sketch=sk)
    assert st == B.SKO_OK, (st, col)
    ref = orth.orth_blocks_one_stage(V, w, intra, Sketch.sparse_sign(64, 8, 5) if intra == "randcholqr" else None)
    check(V, Q.cpu().numpy(), R, ref, e)
    # in place: the same arithmetic on the same columns
    Vi = Vd.t().clone().t()
    Qi, Ri, st, _ = ctx.orth_blocks(Vi, w, Q=Vi, intra=intra, sketch=sk)
    assert st == B.SKO_OK and np.array_equal(R, Ri) and torch.equal(Q, Qi)


def test_one_stage_shifted_buffers(B, ctx):
    """Q one block to the left of V in one buffer: the general schedule, as before."""
    n, w, nb = 3001, 5, 4
    V = wl.glued_blocks(n, nb, w, 3.0)
    buf = torch.empty(((nb + 1) * w, n), dtype=torch.float64, device="cuda").t()
    buf[:, w:].copy_(torch.from_numpy(V))
    sk = B.make_sketch("sparse_sign", 64, 8, 5)
    Q, R, st, col = ctx.orth_blocks(buf[:, w:], w, Q=buf[:, :nb * w], sketch=sk)
    assert st == B.SKO_OK, (st, col)
    check(V, Q.cpu().numpy(), R, orth.orth_blocks_one_stage(V, w, "randcholqr", Sketch.sparse_sign(64, 8, 5)), 3.0)


@pytest.mark.parametrize("e", [10.0, 12.0])
def test_one_stage_ill_conditioned_dependent_blocks(B, ctx, e):
    """Blocks of condition 10^e that also lean on the blocks before them."""
    n, w, nb = 20000, 6, 5
    V = wl.glued_blocks(n, nb, w, e)
    for j in range(1, nb):
        V[:, j * w:(j + 1) * w] = 1e-6 * V[:, j * w:(j + 1) * w] + V[:, (j - 1) * w:j * w]
    Q, R, st, col = ctx.orth_blocks(B.colmajor_from_numpy(V, "cuda"), w, sketch=B.make_sketch("sparse_sign", 64, 8, 5))
    assert st == B.SKO_OK, (st, col)
    Q = Q.cpu().numpy()
    assert metrics.orth_error(Q)[0] <= 1e-13
    assert metrics.backward_error(V, Q, R) <= 1e-14


@pytest.mark.parametrize("w,nb", [(4, 5), (6, 4), (11, 4), (12, 3)])
def test_mixed_look_ahead_matches_block_steps(B, ctx, w, nb):
    n = 5003
    V = B.colmajor_from_numpy(wl.glued_blocks(n, nb, w, 1.0), "cuda", dtype=torch.float32)
    kw = dict(precision="mixed", sketch=B.make_sketch("sparse_sign", 64, 8, 5))
    Q, R, st, _ = ctx.orth_blocks(V, w, **kw)
    assert st == B.SKO_OK
    Qs = torch.empty((nb * w, n), dtype=torch.float32, device="cuda").t()
    Rs = np.zeros_like(R)
    for j in range(nb):
        p = j * w
        _, Rp, Rd, st, _ = ctx.orth_block(Qs[:, :p] if p else None, V[:, p:p + w], Qs[:, p:p + w], **kw)
        assert st == B.SKO_OK
        Rs[p:p + w, p:p + w] = Rd
        if p:
            Rs[:p, p:p + w] = Rp
    # the sums differ by FP64 rounding; a stored value may so round to the next FP32 number
    # (u32 = 2^-24 of its size, in few places)
    assert metrics.rel_diff(R, Rs) <= 1e-9
    assert float((Q - Qs).abs().max()) <= 8 * 2.0 ** -24 * float(Qs.abs().max())


# big panels of 16, 17..33, 48, 60 and 64 columns; 64 columns on 128 exceed the update kernel's LDS
@pytest.mark.parametrize("w,ppb,nb", [(8, 2, 4), (5, 4, 8), (11, 3, 6), (12, 4, 8), (15, 4, 8), (16, 4, 12)])
@pytest.mark.parametrize("n", [1003, 6000])
@pytest.mark.parametrize("reorth", [True, False])
def test_two_stage_panel_widths(B, ctx, w, ppb, nb, n, reorth):
    e = 3.0
    V = wl.glued_blocks(n, nb, w, e)
    Q, R, st, col = ctx.orth_blocks(B.colmajor_from_numpy(V, "cuda"), w, two_stage=True, panels_per_big=ppb,
                                    reorth=reorth, sketch=B.make_sketch("sparse_sign", 128, 8, 2))
    assert st == B.SKO_OK, (st, col)
    ref = orth.orth_blocks_two_stage(V, w, ppb, Sketch.sparse_sign(128, 8, 2), reorth)
    Q = Q.cpu().numpy()
    assert metrics.rel_diff(R, ref.R) <= tol_r(e)
    assert metrics.backward_error(V, Q, R) <= 1e-14
    if reorth:
        assert metrics.orth_error(Q)[0] <= 1e-13


# big panels of 48 columns fuse the update with its Gram matrix, wider FP32 ones do not
@pytest.mark.parametrize("w,ppb,fused", [(12, 4, True), (13, 4, False), (14, 4, False)])
@pytest.mark.parametrize("n", [1003, 6000])
def test_two_stage_mixed_wide_panels(B, ctx, w, ppb, fused, n):
    nb, u32 = 2 * ppb, 2.0 ** -24
    V = wl.glued_blocks(n, nb, w, 1.0)
    Vd = B.colmajor_from_numpy(V, "cuda", dtype=torch.float32)
    ctx.sko_profile_enable(True)
    Q, R, st, col = ctx.orth_blocks(Vd, w, two_stage=True, panels_per_big=ppb, precision="mixed",
                                    sketch=B.make_sketch("sparse_sign", 128, 8, 2))
    names = [s["name"] for s in ctx.sko_profile_read()]
    ctx.sko_profile_enable(False)
    assert st == B.SKO_OK, (st, col)
    assert any(s.startswith("wide_update+gram") for s in names) == fused
    # Q is rounded to FP32 entry by entry: ||I - Q^T Q|| <= 2 u32 ||Q||_F, ||V - Q R||_F <= u32 ||Q||_F ||R||_2 to
    # first order (V_hat and V_bar are rounded once each before it: bounds doubled)
    Q = Q.double().cpu().numpy()
    assert metrics.orth_error(Q)[0] <= 4 * u32 * np.sqrt(nb * w)
    V = Vd.double().cpu().numpy()
    assert np.linalg.norm(V - Q @ R) <= 4 * u32 * np.sqrt(nb * w) * np.linalg.norm(R, 2)
