"""Columns that start at odd elements: the passes read them with the same wide accesses as
aligned ones, so the same block in a buffer with an odd leading dimension and an odd first
element gives bit for bit the same Q and R (same arithmetic, same order of every sum)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2503_16717_amd import workloads as wl  # noqa: E402

pytestmark = pytest.mark.gpu


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


def placed(V, dtype, ld, first):
    """V as a column-major view with leading dimension ld starting `first` elements in."""
    n, N = V.shape
    buf = torch.zeros(first + ld * N, dtype=dtype, device="cuda")
    view = buf.as_strided((n, N), (1, ld), first)
    view.copy_(torch.from_numpy(V).to(dtype))
    return view


@pytest.mark.parametrize("n", [31, 255, 256, 1003, 70001])
@pytest.mark.parametrize("w", [5, 6, 11, 16])
@pytest.mark.parametrize("precision", ["f64", "mixed"])
@pytest.mark.parametrize("scheme", ["one", "two", "gaussian"])
def test_odd_columns_match_aligned(B, ctx, n, w, precision, scheme):
    nb = 4 if n >= 4 * w + 8 else 1
    V = wl.glued_blocks(n, nb, w, 2.0)
    dtype = torch.float64 if precision == "f64" else torch.float32
    kw = dict(precision=precision, sketch=B.make_sketch("sparse_sign", 64, 8, 3))
    if scheme == "two":
        kw.update(two_stage=True, panels_per_big=2 if nb == 4 else 1)
    if scheme == "gaussian":
        th = placed(wl.gaussian_theta(n, 24, 0), torch.float64, n + (n % 2 == 0), 1)
        kw["sketch"] = B.make_sketch("gaussian", theta=th)
    even = (n + 63) // 64 * 64
    odd = n + (n % 2 == 0) + 2
    out = []
    for ld, first in ((even, 0), (odd, 1)):
        Vd = placed(V, dtype, ld, first)
        Q = placed(np.zeros_like(V), dtype, ld, first)
        Q, R, st, col = ctx.orth_blocks(Vd, w, Q=Q, **kw)
        torch.cuda.synchronize()
        assert st == B.SKO_OK, (st, col)
        out.append((Q.double().cpu().numpy(), R))
    assert np.array_equal(out[0][1], out[1][1])
    assert np.array_equal(out[0][0], out[1][0])
