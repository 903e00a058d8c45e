"""The library's host code on a HIP runtime that runs nothing and logs what it
is asked (tests/fake_hip.cpp): which launches, waits and allocations a program
makes.  Each test is a program in a process of its own, which loads that
runtime before libflb.so."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = "/opt/rocm/include"

PRELUDE = """
import ctypes as C, sys
sys.path.insert(0, %r)
sys.modules["torch"] = None  # not needed, and it would bring its own runtime
fake = C.CDLL(%r, C.RTLD_GLOBAL)
fake.fake_log.restype = C.c_char_p
fake.fake_memory.argtypes = [C.c_size_t]
import paper_1204_6734_amd as F
P = F.make_params

def log(kind=None, name=""):
    lines = fake.fake_log().decode().splitlines()
    fake.fake_clear()
    return [x for x in lines if (kind is None or x[0] in kind) and name in x]
"""


@pytest.fixture(scope="session")
def program(tmp_path_factory):
    if shutil.which("g++") is None or not os.path.isdir(ROCM):
        pytest.skip("needs g++ and the HIP headers")
    so = str(tmp_path_factory.mktemp("fake") / "fake_hip.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-Wall",
                    "-D__HIP_PLATFORM_AMD__", "-I", ROCM,
                    os.path.join(ROOT, "tests", "fake_hip.cpp"), "-o", so], check=True)

    def run(code):
        r = subprocess.run([sys.executable, "-c", PRELUDE % (ROOT, so) + code],
                           capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stderr[-4000:]
        return r.stdout

    return run


def test_large_readouts_wait_for_the_steps_before_polling(program):
    """700 closed blocks are more than the small staging area: the steps still
    enqueued are waited for, not polled for, in D2Q9 and D3Q19."""
    program("""
for L in (F.Lattice(P(16, 16, sample_every=1, block_steps=1)),
          F.Lattice3(F.make_params3(8, 4, 4, sample_every=1, block_steps=1))):
    for _ in range(3):  # the large area is taken from the second readout on
        L.step(700)
        log()
        L.covariance()
        lines = log()
        assert not [x for x in lines if x[0] == "P"], lines
        waits = [int(x.split()[2]) for x in lines if x[0] == "S"]
        assert waits[0] > 0, lines
""")


@pytest.mark.parametrize("case", ["readout", "graph"])
def test_another_current_device(program, case):
    """A lattice or ensemble of device 0 used while device 1 is current, as
    programs that hold lattices on several devices do: large readouts, and the
    replayed chunk of an ensemble that advances in two halves."""
    program("""
if %r == "readout":
    L = F.Lattice(P(200, 200))
    fake.hipSetDevice(1)
    for _ in range(3):
        L.populations()
else:
    L = F.Ensemble([P(128, 128, seed=k) for k in range(64)], graph_chunk=10)
    fake.hipSetDevice(1)
    L.step(20)
    assert len({x.split()[1] for x in log("C", "step_kernel")}) == 2
now = C.c_int()
fake.hipGetDevice(C.byref(now))
assert now.value == 1
""" % case)
