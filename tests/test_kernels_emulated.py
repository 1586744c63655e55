"""The kernels of csrc/ built for the host and run lane by lane on the CPU, in orders of the
test's choosing (tests/emulate): what a GPU shows rarely or by a fault is shown here every time."""
import os
import subprocess

import pytest

from paper_2609_36522_amd import build as B

SRC = os.path.join(os.path.dirname(__file__), "emulate")


@pytest.fixture(scope="session")
def emulated(tmp_path_factory):
    """Builds a driver of tests/emulate with the kernel sources; returns a function that runs it."""
    clang = os.path.join(os.path.dirname(os.path.realpath(B.hipcc())), "..", "lib", "llvm", "bin", "clang++")
    out = tmp_path_factory.mktemp("emulate")

    def run(driver, kernels):
        exe = str(out / driver)
        cmd = [clang, "-x", "c++", "-std=c++17", "-O1", "-g", "-pthread", "-Wno-unknown-pragmas", "-I", SRC, "-I", B.INCLUDE,
               "-I", B.CSRC, os.path.join(SRC, driver + ".cpp"), *[os.path.join(B.CSRC, k) for k in kernels], "-o", exe]
        r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
        assert r.returncode == 0, r.stderr[-4000:]
        r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
        assert r.returncode == 0, (r.stdout + r.stderr)[-4000:]
        return r.stdout

    return run


def test_blocks_of_a_fused_sweep_leave_whole(emulated):
    assert "fused exit ok" in emulated("fused_exit", ["k_solver.hip", "k_epsnet.hip"])


def test_rows_of_fine_partial_outputs(emulated):
    assert "fine rows ok" in emulated("fine_rows", [])
