"""The wide path's cooperative run (fw_wide_run.hip) in a CPU emulation of the device, a process per
workgroup: bit for bit the launch-by-launch run, and, with a workgroup that never starts, every wait
gives up and the log launch leaves the counts alone (it would index them with decisions that
were never written)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def build(tmp_path_factory):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("g++ not available")
    d = tmp_path_factory.mktemp("wide_run_emu")

    def make(limit):
        exe = str(d / f"emu{limit}")
        if not os.path.exists(exe):
            subprocess.check_call([gxx, "-std=c++20", "-O2", f"-DFW_POLL_LIMIT={limit}", "-I", os.path.join(HERE, "emu", "shim"),
                                   "-I", os.path.join(ROOT, "include"), "-o", exe, os.path.join(HERE, "emu", "emu_wide_run.cpp"),
                                   "-lpthread"])
        return exe
    return make


def run(exe, *args):
    return subprocess.run([exe, *map(str, args)], capture_output=True, text=True, timeout=300, check=True).stdout.strip()


@pytest.mark.parametrize("ns,rows,d,N,R,T,M,steps", [
    (4, 0, 300, 25, 1, 4, 1, 3), (2, 0, 132, 7, 2, 3, 2, 8), (2, 3, 500, 13, 1, 3, 1, 2), (2, 3, 260, 5, 1, 4, 3, 8)])
def test_same_bits(build, ns, rows, d, N, R, T, M, steps):
    assert run(build(1 << 20), ns, rows, d, N, R, T, M, steps, -1) == "same"


@pytest.mark.parametrize("rows", [0, 3])
def test_missing_workgroup(build, rows):
    assert run(build(64), 2, rows, 260, 5, 1, 2, 1, 2, 1) == "gave up, counts untouched"
