"""Host bookkeeping of a population where a device allocation is refused, with
the HIP runtime replaced by a stand-in that counts allocations (hip_stub.cpp):
the library's own code runs, no kernel does and no GPU is needed."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
LIBRARY = os.path.join(os.path.dirname(HERE), "paper_2405_00698_amd", "_lib.py")

PRELUDE = """
import ctypes as C, importlib.util, os, sys
stub = C.CDLL(sys.argv[1], mode=os.RTLD_GLOBAL | os.RTLD_NOW)
spec = importlib.util.spec_from_file_location("lib", sys.argv[2])
lib = importlib.util.module_from_spec(spec)
spec.loader.exec_module(lib)
L = lib.load()
some = C.c_void_p(64)  # stands for a caller's device array; nothing reads it

def population(sides, params=None):
    h = C.c_void_p()
    p = params or lib.default_params()
    assert L.pop_create(C.byref(p), len(sides), (C.c_int32 * len(sides))(*sides), None, C.byref(h)) == 0
    return h

def built(sides, params=None):
    h = population(sides, params)
    assert L.pop_build_from_voxels(h, some, some) == 0
    return h

def recorded(h, every, steps):
    return L.pop_reset(h) or L.pop_record(h, every, steps) or L.pop_step(h, steps)

def backward(h):
    return L.pop_backward(h, some, some, some, some, None, None, None)

def destroyed(h):
    assert L.pop_destroy(h) == 0
    assert stub.stub_bad_frees() == 0, "freed twice: %d" % stub.stub_bad_frees()
    assert stub.stub_bad_grids() == 0, "launches beyond a grid's size: %d" % stub.stub_bad_grids()
    assert stub.stub_live() == 0, "left allocated: %d" % stub.stub_live()
"""


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    so = tmp_path_factory.mktemp("stub") / "hip_stub.so"
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", os.path.join(HERE, "hip_stub.cpp"), "-o",
                           str(so)])
    return str(so)


def run(stub, body):
    r = subprocess.run([sys.executable, "-c", PRELUDE + body, stub, LIBRARY], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr


def test_refused_population_does_not_fail_the_next(stub):
    """pop_create is refused at any one of its allocations, and so are the
    checkpoints of pop_record: the next calls work."""
    run(stub, '''
stub.stub_fail(-1, -1)
destroyed(built([5, 8, 12]))
total = stub.stub_mallocs()
assert total >= 20
for n in range(total):
    h, p = C.c_void_p(), lib.default_params()
    stub.stub_fail(n, n + 1)
    assert L.pop_create(C.byref(p), 3, (C.c_int32 * 3)(5, 8, 12), None, C.byref(h)) == lib.SR_ENOMEM, n
    stub.stub_fail(-1, -1)
    assert stub.stub_live() == 0, n
    destroyed(built([5, 8, 12]))
for n in range(2):
    h = built([5, 8, 12])
    stub.stub_fail(n, n + 1)
    assert L.pop_record(h, 10, 40) == lib.SR_ENOMEM
    assert recorded(h, 10, 40) == 0, (n, L.sr_last_error())
    destroyed(h)
''')


@pytest.mark.parametrize("sides", [[5, 5], [8, 12], [4, 6, 9]])
@pytest.mark.parametrize("model", ["default", "table2"])
def test_refused_adjoint_scratch(stub, sides, model):
    """Growing the reverse sweep's scratch is refused at any one of its
    allocations: the call reports it, and the population goes on, with a smaller
    interval, the larger one once there is memory, or its end."""
    run(stub, "sides, model = %r, %r\n" % (sides, model) + '''
params = lib.table2_params() if model == "table2" else None
h = built(sides, params)
assert recorded(h, 10, 40) == 0
stub.stub_fail(-1, -1)
assert backward(h) == 0
total = stub.stub_mallocs()  # the scratch and the time table
assert total >= 13
destroyed(h)
for after in ("smaller", "same", "destroy"):
    for n in range(total - 1):
        h = built(sides, params)
        assert recorded(h, 10, 40) == 0 and backward(h) == 0
        assert recorded(h, 20, 40) == 0
        stub.stub_fail(n, n + 1)
        assert backward(h) == lib.SR_ENOMEM, n
        stub.stub_fail(-1, -1)
        if after == "smaller":
            assert recorded(h, 5, 40) == 0 and backward(h) == 0, (n, L.sr_last_error())
        elif after == "same":
            assert backward(h) == 0, (n, L.sr_last_error())
        destroyed(h)
''')


@pytest.mark.parametrize("build", ["pop_build_from_voxels(h, some, some)", "pop_build_from_genomes(h, some, some, 0)"])
def test_refused_counts_buffer(stub, build):
    """The first build is refused its host buffer: it says so, and a later one works."""
    run(stub, "build = lambda h: L.%s\n" % build + '''
h = population([5, 8])
stub.stub_fail_pinned(1)
assert build(h) == lib.SR_ENOMEM
assert L.pop_step(h, 1) == lib.SR_ESTATE
stub.stub_fail_pinned(0)
assert build(h) == 0 and L.pop_step(h, 1) == 0, L.sr_last_error()
destroyed(h)
''')


@pytest.mark.parametrize("precision", [0, 1])
def test_population_beyond_a_grid_row(stub, precision):
    """70,000 robots: every launch of a generation stays within a grid."""
    run(stub, "precision = %d\n" % precision + '''
h = population([2] * 70000)
assert L.pop_build_from_genomes(h, some, some, precision) == 0 and recorded(h, 10, 20) == 0 and backward(h) == 0
destroyed(h)
''')


def test_rebuild_takes_up_the_voxel_kernel_again(stub):
    """pop_set_spring_params replaces the kernels that rebuild the parameters
    from voxels until the next build, unless another kernel was chosen since."""
    run(stub, '''
VOX = 96
def variant(h, n):
    b, v = C.c_int32(), C.c_int32()
    assert L.pop_get_persist_variant(h, n, C.byref(b), C.byref(v)) == 0
    return b.value, v.value
def configs(n):
    b, v = (C.c_int32 * 64)(), (C.c_int32 * 64)()
    return [(b[i], v[i]) for i in range(L.sr_persist_configs(n, b, v, 64))]
for params, n in ((lib.table2_params(), 12), (lib.default_params(), 11), (lib.default_params(), 5)):
    dash = params.zeta_spring != 0
    vox = [c for c in configs(n) if bool(c[1] & 16) == dash and c[1] & VOX]
    plane = [c for c in configs(n) if bool(c[1] & 16) == dash and not c[1] & VOX]
    for own in [None] + vox:
        h = built([5, n, n], params)
        if own:
            assert L.pop_set_persist_variant(h, n, *own) == 0
        before = variant(h, n)
        assert L.pop_set_spring_params(h, some, some, some) == 0 and L.pop_step(h, 3) == 0
        assert not variant(h, n)[1] & VOX
        assert L.pop_build_from_voxels(h, some, some) == 0 and L.pop_step(h, 3) == 0
        assert variant(h, n) == before, (n, own)
        # a kernel chosen after the parameters stays
        assert L.pop_set_spring_params(h, some, None, None) == 0
        assert L.pop_set_persist_variant(h, n, *plane[-1]) == 0
        assert L.pop_build_from_voxels(h, some, some) == 0
        assert variant(h, n) == plane[-1]
        destroyed(h)
''')


@pytest.mark.parametrize("sides,lanes", [([8, 8], 3), ([5, 12], 4), ([4, 5, 6, 7, 8], 4)])
def test_recording_makes_the_streams_it_uses(stub, sides, lanes):
    """A stream costs the first recording of a population about 80 us."""
    run(stub, "sides, lanes = %r, %d\n" % (sides, lanes) + '''
h = built(sides)
before = stub.stub_streams()
assert L.pop_record(h, 10, 40) == 0
assert stub.stub_streams() - before == lanes
assert L.pop_step(h, 40) == 0 and backward(h) == 0 and recorded(h, 10, 40) == 0
assert stub.stub_streams() - before == lanes
destroyed(h)
''')


def test_only_graphs_of_one_launch_a_lane_are_captured(stub):
    """Several launches on a lane beside other lanes go out directly; a single
    side, the per-step form and one launch a lane are captured once per length."""
    run(stub, '''
def captured(h, *lengths):
    before = stub.stub_captures()
    for n in lengths:
        assert L.pop_step(h, n) == 0
    return stub.stub_captures() - before
def schedule(h, sides, lanes):
    n = len(sides)
    assert L.pop_set_schedule(h, n, (C.c_int32 * n)(*sides), (C.c_int32 * n)(*lanes)) == 0
AUTO, PLAIN = 0, 2
h = built([5, 8, 12, 5])
assert captured(h, 100, 100, 30) == 2              # the default: a lane for each side
assert L.pop_set_step_config(h, AUTO, 0, 50) == 0
assert captured(h, 100, 51) == 0                   # several launches a call
assert captured(h, 50, 20) == 2
assert L.pop_set_step_config(h, AUTO, 0, 0) == 0
schedule(h, [12, 8, 5], [0, 1, 0])
assert captured(h, 100, 30) == 0                   # two sides on a lane
schedule(h, [12, 8, 5], [2, 0, 1])
assert captured(h, 100) == 1
schedule(h, [12, 8, 5], [0, 0, 0])
assert L.pop_set_step_config(h, PLAIN, 0, 0) == 0
assert captured(h, 10) == 1
destroyed(h)
h = built([6, 6])
assert L.pop_set_step_config(h, AUTO, 0, 25) == 0
assert captured(h, 100) == 1                       # one lane: a chain
assert L.pop_set_graphs(h, 0) == 0
assert captured(h, 100) == 0
destroyed(h)
''')
