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


@pytest.mark.parametrize("other", ["ensemble", "lattice", "d3q19", "server"])
def test_two_graph_branches_only_while_nothing_else_is_at_work(program, other):
    """An ensemble that fills the chip replays two branches alone, one while
    another object has work that was not waited for, and two again after."""
    program("""
def ensemble():
    return F.Ensemble([P(128, 128, seed=k, sample_every=5) for k in range(64)], graph_chunk=10)

class Server:  # at work between a failed chunk and its end
    def __init__(self):
        self.S = F.Server(1 << 28, threaded=False, chunk_steps=4)
        self.S.submit(P(64, 64), 8)
    def step(self, n):
        fake.fake_fail(b"step_kernel", 3)
        try:
            self.S.pump(1)
            raise SystemExit("no failure")
        except F.FlbError:
            pass
    def sync(self):
        self.S.pump(1)

E = ensemble()
O = {"ensemble": ensemble, "lattice": lambda: F.Lattice(P(64, 64)), "server": Server,
     "d3q19": lambda: F.Lattice3(F.make_params3(8, 8, 8))}[%r]()

def branches():
    log()
    E.step(20)
    return [int(x.split()[2]) for x in log("G")]

assert branches() == [2, 2]
O.step(10)
if %r == "ensemble":
    assert [x.split()[2] for x in log("G")] == ["1"]  # E is still at work
assert branches() == [1, 1]
O.sync()
assert branches() == [1, 2] and not log("C")  # alone at two replays
O.step(10)
del O
assert branches() == [2, 2]
""" % (other, other))


@pytest.mark.parametrize("prec,n,branches", [("FP32_SHIFTED", 255, 1), ("FP32_SHIFTED", 256, 2),
                                             ("FP64", 127, 1), ("FP64", 128, 2)])
def test_populations_beyond_the_cache_take_two_branches_beside_other_work(program, prec, n,
                                                                          branches):
    program("""
E = F.Ensemble([P(128, 128, seed=k, precision=F.%s) for k in range(%d)], graph_chunk=10)
L = F.Lattice(P(64, 64))
L.step(10)
E.step(10)
assert [x.split()[2] for x in log("G")] == ["%d"]
""" % (prec, n, branches))


def test_a_server_takes_two_streams_only_alone(program):
    program("""
S = F.Server(1 << 30, threaded=False, chunk_steps=4)
for k in range(40):
    S.submit(P(128, 128, seed=k), 12)
L = F.Lattice(P(64, 64))

def streams():
    log()
    S.pump(1)
    return len({x.split()[1] for x in log("K", "step_kernel")})

assert streams() == 2
L.step(1)
assert streams() == 1
L.sync()
assert streams() == 2
""")


@pytest.mark.parametrize("nx,n,kw,second", [
    (64, 1, dict(), True), (64, 1, dict(sample_every=1), True),
    # sums of every step, where only steps without are taken together
    (256, 1, dict(), True), (256, 1, dict(sample_every=1), False),
    (256, 1, dict(sample_every=4), False), (256, 1, dict(sample_every=5), True),
    (256, 1, dict(sk_every=5), True), (256, 1, dict(sk_every=4), False),
    (3072, 1, dict(), True), (3072, 1, dict(sample_every=4), False),
    (3072, 1, dict(sample_every=5), True), (3072, 1, dict(sample_every=1 << 30), True),
    (160, 64, dict(basis=1), True), (160, 64, dict(basis=1, sample_every=2), False),
    (160, 64, dict(basis=1, sample_every=5), True),
    # strips that use four fifths of their lanes: 360 and 450 MiB
    (256, 160, dict(), False), (256, 200, dict(), True), (256, 200, dict(sample_every=5), False),
    (256, 200, dict(sample_every=10), True),
])
def test_second_buffers_only_where_they_are_used(program, nx, n, kw, second):
    """A group allocates its populations twice exactly where launches of
    several steps are made (the period of the sampling is stepped through)."""
    program("""
nx, n, kw = %d, %d, dict(%r)
log()
ps = [P(nx, nx, seed=k, **kw) for k in range(n)]
L = F.Ensemble(ps) if n > 1 else F.Lattice(ps[0])
big = max(int(x.split()[1]) for x in log("M"))
pops = n * F.population_bytes(ps[0])
L.step(40)
several = log("K", "step_m")
assert bool(several) == %r, several[:3]
# one lattice needs what bytes_needed says and the second buffer; the members
# of these ensembles take less than their populations beside them
need = F.Lattice.bytes_needed(ps[0]) if n == 1 else 2 * pops
assert (big > need) == %r and big < need + pops + 4096, (big, need, pops)
""" % (nx, n, kw, second, second))


@pytest.mark.parametrize("every,branches", [(0, 1), (1, 2), (2, 2), (5, 1), (10, 1)])
def test_branches_where_a_chunk_holds_no_passes(program, every, branches):
    program("""
E = F.Ensemble([P(160, 160, basis=F.BASIS_HERMITE, seed=k, sample_every=%d) for k in range(64)],
               graph_chunk=20)
E.step(20)
assert [x.split()[2] for x in log("G")] == ["%d"]
""" % (every, branches))


@pytest.mark.parametrize("nx,ny,n,tiles,tiles_summed", [
    (256, 99, 350, 99, 100),  # 304 MiB: 256 x 1 tiles without sums, 64 x 4 with
    (256, 99, 290, 100, 100),  # 252 MiB
    (257, 99, 350, 125, 125),  # 256 x 1 tiles would be mostly empty
    (256, 257, 150, 257, 257),  # more than 65536 sites: 256 x 1 throughout
])
def test_tile_shapes_of_ensembles_beyond_the_cache(program, nx, ny, n, tiles, tiles_summed):
    program("""
E = F.Ensemble([P(%d, %d, seed=k, ux0=0.3 if k < 20 else 0.0, sample_every=4)
                for k in range(%d)])
n = len(E.params)
E.set_launch(1, 0)
log()
E.step(2)
grids = [int(x.split()[3]) for x in log("K", "step_kernel")]
want = [%d, %d]  # the step with sums comes first; two compute classes
assert grids == [(n - 20) * want[0], 20 * want[0], (n - 20) * want[1], 20 * want[1]], grids
""" % (nx, ny, n, tiles_summed, tiles))


def test_a_full_device_holds_nearly_as_many_small_lattices(program):
    """A program that fills the device gives second buffers a sixteenth of it at
    most."""
    program("""
one = F.Lattice.bytes_needed(P(64, 64))  # a lattice that takes a second buffer
total = 400 * one
fake.fake_memory(total)
held = []
try:
    while True:
        held.append(F.Lattice(P(64, 64)))
except F.FlbError as e:
    assert e.code == F.E_OOM
assert len(held) >= 400 * 15 // 16, len(held)
assert sum(int(x.split()[1]) > one + one // 4 for x in log("M")) > 5
""")


def test_second_buffers_beside_other_memory(program):
    """Memory that something else holds does not take the launches of several
    steps from a lattice, and lattices that fill the rest of it are nearly as many
    as without second buffers; those of destroyed lattices no longer count."""
    program("""
total = 288 << 30
other = C.c_void_p()
fake.hipMalloc.argtypes = [C.c_void_p, C.c_size_t]
fake.hipFree.argtypes = [C.c_void_p]
small, large = P(64, 64), P(8192, 8192)  # the larger one: 2.25 GiB

def several(p):
    L = F.Lattice(p)
    L.step(4)
    return L.pass_steps() == 4, L

assert fake.hipMalloc(C.byref(other), int(0.9 * total)) == 0
assert several(small)[0]
assert not several(large)[0]  # of 28.8 GiB
fake.hipFree(other)
for _ in range(2):
    held = [several(large) for _ in range(9)]
    assert [h[0] for h in held] == [True] * 7 + [False] * 2, [h[0] for h in held]
    held.pop(0)
    assert several(large)[0]
    del held

one = F.Lattice.bytes_needed(small)
assert fake.hipMalloc(C.byref(other), total - 400 * one) == 0
held = []
try:
    while True:
        held.append(F.Lattice(small))
except F.FlbError as e:
    assert e.code == F.E_OOM
assert len(held) >= 400 * 15 // 16, len(held)
""")


@pytest.mark.parametrize("launch", [1, 2, 5])
def test_a_failed_chunk_leaves_nothing_on_the_second_stream(program, launch):
    """The next chunk writes the tables that the second stream's launches of
    the failed one read."""
    program("""
S = F.Server(1 << 30, threaded=False, chunk_steps=4)
for k in range(40):
    S.submit(P(128, 128, seed=k), 12)
S.pump(1)
second = {x.split()[1] for x in log("K", "step_kernel")}
assert len(second) == 2
fake.fake_fail(b"step_kernel", %d)
try:
    S.pump(1)
    raise SystemExit("no failure")
except F.FlbError:
    pass
lines = [x for x in log("KS") if x[0] == "S" or "step_kernel" in x]
for s in sorted(second)[1:]:  # the second stream is the later one
    last = [x[0] for x in lines if x.split()[1] == s]
    assert last == [] or last[-1] == "S", lines
""" % launch)


def test_pass_steps_counts_launches_of_several_steps(program):
    program("""
for chunk in (0, 12):
    L = F.Lattice(P(64, 64, sample_every=3, block_steps=5))
    L.set_graph_chunk(chunk)
    E = F.Ensemble([P(32, 30, seed=k) for k in range(4)], graph_chunk=chunk)
    for G in (L, E):
        total = 0
        for n in (1, 7, 24, 5, 36):
            G.step(n)
            total += n
            assert 0 <= G.pass_steps() <= total
        assert G.pass_steps() > total // 2
        before = G.pass_steps()
        G.set_launch(1, 0)
        G.step(40)
        assert G.pass_steps() == before
S = F.Lattice(P(64, 64, sample_every=1, block_steps=1))  # every step closes a block
S.step(20)
assert S.pass_steps() == 0
L = F.Lattice(P(64, 64))
log()
L.step(41)
assert len(log("K", "step_kernel")) == 41 - L.pass_steps()
try:
    F._check(F.load().flb_lattice_pass_steps(L.h, None), "")
    raise SystemExit("accepted")
except F.FlbError as e:
    assert e.code == F.E_ARG
assert F.load().flb_ensemble_pass_steps(None, None) == F.E_ARG
""")
