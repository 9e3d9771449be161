"""Device memory that the runtime refuses: the call that can do with less goes on, the others report
SKO_ENOMEM, and neither leaves the runtime's error for a later call to trip over.  A host program
(alloc_refused.cpp) refuses the library's requests itself, so no memory is exhausted."""
import os
import subprocess

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
PKG = os.path.join(ROOT, "paper_2503_16717_amd")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    exe = str(tmp_path_factory.mktemp("alloc") / "alloc_refused")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", f"-I{ROCM}/include", f"-I{ROOT}/include",
                    f"-I{PKG}/csrc", os.path.join(HERE, "alloc_refused.cpp"), "-o", exe, os.path.join(PKG, "libsko.so"),
                    f"-L{ROCM}/lib", "-lamdhip64", f"-Wl,-rpath,{PKG}:{ROCM}/lib"], check=True)
    return exe


def run(program, *mode):
    r = subprocess.run([program, *mode], capture_output=True, text=True, timeout=60)
    print(r.stdout, r.stderr, flush=True)
    assert r.returncode == 0
    return {k: int(v) for k, v in (line.split() for line in r.stdout.splitlines())}


SKO_OK, SKO_ENOMEM = 0, 3


@pytest.mark.parametrize("mode", [("gmres",), ("gmres", "jacobi"), ("batch",)])
def test_solve_without_room_for_the_diagonals_runs_on_csr(program, mode):
    got = run(program, *mode)
    assert got == dict(status=SKO_OK, refused=1, converged=1, diagonals=0, left_error=0)


def test_refused_call_leaves_the_next_one_alone(program):
    got = run(program, "every")
    assert got == dict(refused_status=SKO_ENOMEM, status=SKO_OK, status_plain=SKO_OK, same_r=1, left_error=0)


def test_blocks_without_room_to_look_ahead_go_one_by_one(program):
    got = run(program, "blocks")
    assert got == dict(status=SKO_OK, refused=1, status_plain=SKO_OK, same_r=1, left_error=0)


def test_autotuner_scratch(program):
    """Scratch of 2 w + p_max = 30 columns (the rest: partial sums of 8 workgroups per compute unit)."""
    got = run(program, "autotune")
    assert got["tune_one_stage"] == SKO_OK and 30 <= got["doubles_per_row"] <= 33


def test_autotuner_kinds(program):
    """The look-ahead's passes, and those of the same shapes taken one block or panel at a time."""
    got = run(program, "autotune")
    del got["doubles_per_row"]
    assert got == dict(tune_one_stage=SKO_OK, block_steps=6, look_ahead=3, tune_two_stage=SKO_OK, panels=5)
