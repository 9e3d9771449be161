"""Resources of the compiled pass kernels that their times depend on: where a row solve keeps its
diagonal's reciprocals (static LDS of W doubles per solve, or registers)."""
import ctypes as C

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


class PassKey(C.Structure):
    _fields_ = [("W", C.c_int), ("f32", C.c_bool), ("red", C.c_int), ("upd", C.c_bool), ("ntrsm", C.c_int),
                ("write", C.c_bool), ("tiles", C.c_int), ("panel", C.c_int), ("pair", C.c_int)]


class FuncAttributes(C.Structure):
    _fields_ = [("binary", C.c_int), ("cache", C.c_int), ("const_bytes", C.c_size_t), ("local_bytes", C.c_size_t),
                ("max_dynamic_lds", C.c_int), ("max_threads", C.c_int), ("registers", C.c_int), ("carveout", C.c_int),
                ("ptx", C.c_int), ("lds_bytes", C.c_size_t)]


@pytest.mark.parametrize("W", range(8, 17))
@pytest.mark.parametrize("upd", [False, True])
@pytest.mark.parametrize("f32,panel", [(False, 0), (True, 0), (True, 2)])
def test_reciprocals_of_a_single_solve(W, upd, f32, panel):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_16717_amd import binding as B
    torch.zeros(1, device="cuda")
    lib = C.CDLL(B._LIB_PATH)
    kernel = lib["_ZN3sko14pass_kernel_idERKNS_7PassKeyE"]
    kernel.restype = C.c_void_p
    fn = kernel(C.byref(PassKey(W, f32, 0, upd, 1, True, 0, panel, 0)))
    attr = FuncAttributes()
    assert lib["hipFuncGetAttributes"](C.byref(attr), C.c_void_p(fn)) == 0
    in_lds = W >= 9 and not (upd and W >= 10)
    assert (attr.lds_bytes >= 8 * W) == in_lds, (attr.lds_bytes, attr.registers)
    assert attr.local_bytes == 0
