"""The library's host code on a machine without a GPU: which work it enqueues where, what
it allocates and what it does when a call fails.  Each test runs the built library in a
process of its own over fake_hip.cpp, a HIP runtime that notes every call, does copies at
once and runs no kernel, so nothing here says what a kernel computes."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))

PRELUDE = """
import ctypes, re, sys, threading
sys.modules["torch"] = None  # it would load the real runtime
fail_new = ctypes.CDLL({new!r}, ctypes.RTLD_GLOBAL)
fake = ctypes.CDLL({lib!r}, ctypes.RTLD_GLOBAL)
fake.fake_reset.argtypes = [ctypes.c_size_t]
fake.fake_capture.argtypes = [ctypes.c_void_p, ctypes.c_int]
fake.fake_fail.argtypes = [ctypes.c_char_p, ctypes.c_int]
fake.fake_notes.restype = ctypes.c_char_p
fake.fake_used.restype = fake.fake_allocs.restype = ctypes.c_size_t
sys.path.insert(0, {root!r})
import numpy as np
from paper_2609_16361_amd import binding, inputs
F32, F16 = binding.LBM_STORE_F32, binding.LBM_STORE_F16

def notes(what=""):
    "The calls noted since the last reset: (what, stream, thread, rest), of kind `what`."
    out = []
    for line in fake.fake_notes().decode().splitlines():
        w, s, t, rest = line.split(" ", 3)
        if not what or w == what:
            out.append((w, int(s.split("=")[1], 16), int(t.split("=")[1]), rest))
    return out

def kernels():
    "The launched kernels by name: k_step, k_step_pair, ..."
    out = []
    for n in notes("launch"):
        m = re.search(r"(\\d{{1,2}})(k_\\w+)", n[3])  # a mangled name: its length comes first
        out.append(m.group(2)[:int(m.group(1))])
    return out

def value(rest, key):
    return int(re.search(key + "=([0-9a-f]+)", rest).group(1), 16)

def case(dims, **kw):
    return inputs.random_smooth(*dims, seed=3, amp=0.03, **kw)

def status(fn):
    try:
        fn()
    except binding.LbmError as e:
        return e.status
    return 0

fake.fake_reset(1 << 33)
"""


@pytest.fixture(scope="session")
def run(tmp_path_factory):
    at = tmp_path_factory.mktemp("fake")
    lib, new = str(at / "libfake_hip.so"), str(at / "libfail_new.so")
    cc = ["g++", "-std=c++17", "-O1", "-shared", "-fPIC", os.path.join(HERE, "fake_hip.cpp")]
    # its own allocations do not fail: it holds its own operator new
    subprocess.run(cc + ["-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-Wl,-soname,libamdhip64.so.7", "-Wl,-Bsymbolic",
                         "-static-libstdc++", "-Wl,--exclude-libs,ALL", "-o", lib, "-lpthread"], check=True)
    subprocess.run(cc + ["-DFAIL_NEW", "-o", new], check=True)

    def go(code):
        prelude = PRELUDE.format(lib=lib, new=new, root=os.path.dirname(HERE))
        r = subprocess.run([sys.executable, "-c", prelude + code], capture_output=True, text=True, timeout=300)
        assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]

    return go


def test_copies_on_the_per_thread_stream_stay_in_the_callers_thread(run):
    # handle 2 means another stream in every thread: what a worker enqueued there would
    # not be ordered after the caller's kernels
    run("""
c = case((96, 64, 40))
with binding.Solver(c.params, stream=2) as s, binding.Batch(1 << 26, stream=2) as b:
    s.init(c.Q0)
    s.step(3)
    f, _ = s.populations()
    s.moments()
    s.set_populations(f, 3)
    i = b.add(c.params, c.Q0, 5)
    b.populations(i)
    b.moments(i)
assert len(notes("copy")) > 30
assert all(t == 0 for _, _, t, _ in notes("copy"))
fake.fake_reset(0)
with binding.Solver(c.params) as s:  # on any other stream the workers share the copies
    s.init(c.Q0)
assert {t for _, _, t, _ in notes("copy")} == {0, 1, 2, 3}
""")


def test_captured_batch_steps_are_single_and_stay_so(run):
    # a graph of the caller's must not keep the second arena's address, which can be given
    # up, nor passes of several steps, which check an instance's end once per pass
    run("""
with binding.Batch(1 << 26, graph_steps=64) as b:
    for d, st in (((40, 36, 33), F32), ((300, 4, 4), F32), ((300, 4, 4), F16)):
        c = case(d)
        b.add(c.params, c.Q0, 1000, storage=st)
    b.run(10)
    assert {"k_batch_pair", "k_batch_tube"} <= set(kernels())
    stream = notes("launch")[-1][1]
    fake.fake_reset(0)
    fake.fake_capture(stream, 1)
    b.run(10)
    assert set(kernels()) == {"k_batch_step", "k_batch_advance"}, set(kernels())
    fake.fake_capture(stream, 0)
    fake.fake_reset(0)
    b.run(64)
    assert set(kernels()) == {"k_batch_step", "k_batch_advance"}, set(kernels())
""")


@pytest.mark.parametrize("dims,kernel", [((40, 36, 33), b"k_step_pair"), ((300, 4, 4), b"k_step_tube")])
@pytest.mark.parametrize("after", [0, 1, 2])
def test_a_failed_pass_leaves_no_state_to_go_on_from(run, dims, kernel, after):
    # 15 and 39 steps: an even step into the second buffer and seven pairs; four passes of
    # a tube.  Only a tube's first pass leaves the state where it was.
    run(f"""
c = case({dims})
with binding.Solver(c.params) as s:
    s.init(c.Q0)
    fake.fake_fail({kernel!r}, {after})
    assert status(lambda: s.step(15 if {kernel!r} == b"k_step_pair" else 39)) == binding.LBM_EDEVICE
    kept = {after} == 0 and {kernel!r} == b"k_step_tube"
    for call in (lambda: s.step(1), s.moments, s.populations):
        assert status(call) == (0 if kept else binding.LBM_ESTATE)
    s.init(c.Q0)
    s.step(39)
    s.moments()
""")


@pytest.mark.parametrize("kernel,after,kept", [(b"k_batch_tube", 0, True), (b"k_batch_tube", 1, False),
                                               (b"k_batch_pair", 0, False)])
def test_a_failed_pass_ends_a_batch(run, kernel, after, kept):
    run(f"""
with binding.Batch(1 << 26, graph_steps=64) as b:
    c = case((40, 36, 33) if {kernel!r} == b"k_batch_pair" else (300, 4, 4))
    i = b.add(c.params, c.Q0, 1000)
    fake.fake_fail({kernel!r}, {after})
    assert status(lambda: b.run(30)) == binding.LBM_EDEVICE
    for call in (lambda: b.run(1), lambda: b.moments(i), lambda: b.populations(i), b.nonfinite):
        assert status(call) == (0 if {kept} else binding.LBM_ESTATE)
    b.remove(i)
""")


def test_no_call_waits_for_the_device(run):
    # other streams' work is none of a context's business, whatever the size of its state
    run("""
for storage, dims in ((F32, (128, 128, 72)), (F16, (128, 128, 130))):  # 165 and 149 MB of state
    c = case(dims)
    with binding.Solver(c.params, storage=storage) as s:
        s.init(c.Q0)
        s.step(5)
        s.moments()
assert binding.lbm_state_bytes(s.cparams) >= 128 << 20
assert len(notes("sync")) > 4 and not notes("device-sync")
""")


def test_batch_runs_of_odd_length_upload_nothing_and_stay_fast(run):
    run("""
with binding.Batch(1 << 26, graph_steps=64) as b:
    for d, st in (((40, 36, 33), F32), ((300, 4, 4), F32), ((300, 4, 4), F16), ((24, 24, 24), F16)):
        c = case(d)
        b.add(c.params, c.Q0, 1000, storage=st)
    b.run(1)
    fake.fake_reset(0)
    for n in (1, 3, 7, 9, 1, 15):
        b.run(n)
    assert not notes("copy") and not notes("sync") and not notes("malloc")
    fake.fake_reset(0)
    b.run(9)  # from an odd step: one single step, then fast ones
    assert kernels()[:3] == ["k_batch_step", "k_batch_step", "k_batch_advance"]  # a group each for FP32 and FP16
    assert {"k_batch_pair", "k_batch_tube"} <= set(kernels())
    # a later and smaller instance does not take the others out of fast runs
    b.run(1)
    c = case((50, 3, 3))
    b.add(c.params, c.Q0, 1000)
    fake.fake_reset(0)
    b.run(21)
    assert {"k_batch_pair", "k_batch_tube"} <= set(kernels())
""")


def test_second_buffers_are_taken_by_the_first_steps_that_use_them(run):
    run("""
grid, tube = case((40, 36, 33)), case((300, 4, 4))
S = ctypes.create_string_buffer(5 * 4 * grid.cells)
def held(s):
    return s.passes()["second_bytes"]
with binding.Solver(grid.params) as s:
    n = fake.fake_allocs()
    assert n == 2 and held(s) == 0  # the populations and the diagnostic ring
    binding.lbm_init_fields_device(s.ctx, np.ascontiguousarray(grid.Q0).ctypes.data)
    s.step(2)
    s.step(40, 1)
    s.step(40, 2)
    s.set_source(ctypes.addressof(S))
    s.step(8)
    s.set_source(None)
    stream = notes("launch")[-1][1]
    fake.fake_capture(stream, 1)
    s.step(8)
    fake.fake_capture(stream, 0)
    s.autotune(4)
    assert held(s) == 0 and s.passes()["passes"] == s.passes()["steps"]
    before = s.passes()
    s.step(9)
    assert held(s) == binding.lbm_state_bytes(s.cparams)
    after = s.passes()
    assert after["steps"] - before["steps"] == 9 and after["passes"] - before["passes"] == 5
with binding.Solver(grid.params) as s:
    s.init(grid.Q0)  # staged there, and the steps to come use it
    assert held(s) > 0
for kw in (dict(odd_lds=False), dict(passes=False), dict(storage=F16)):
    with binding.Solver(grid.params, **kw) as s:
        s.init(grid.Q0)
        s.step(20)
        assert held(s) == 0 and s.passes() == dict(steps=20, passes=20, second_bytes=0)
with binding.Batch(1 << 26) as b:
    b.add(grid.params, grid.Q0, 100, storage=F16)
    b.run(20)
    assert b.passes() == dict(steps=20, fast_steps=0, second_bytes=0)
    b.add(tube.params, tube.Q0, 100, storage=F16)
    b.run(20)
    assert b.passes() == dict(steps=40, fast_steps=20, second_bytes=1 << 26)
assert fake.fake_used() == 0
""")


def test_second_buffers_can_be_declined_and_given_back(run):
    run("""
c = case((40, 36, 33))
with binding.Solver(c.params) as s, binding.Batch(1 << 26) as b:
    s.init(c.Q0)
    i = b.add(c.params, c.Q0, 1000)
    own = fake.fake_used()
    for _ in range(2):
        s.step(21)
        b.run(20)
        full = fake.fake_used()
        assert s.passes()["second_bytes"] > 0 and b.passes()["second_bytes"] == 1 << 26
        s.set_passes(False)
        b.set_passes(False)
        assert fake.fake_used() == full - binding.lbm_state_bytes(s.cparams) - (1 << 26)
        fake.fake_reset(0)
        s.step(21)
        b.run(20)
        s.moments()
        b.moments(i)
        assert not {"k_step_pair", "k_step_even_to", "k_batch_pair"} & set(kernels())
        assert s.passes()["second_bytes"] == b.passes()["second_bytes"] == 0
        s.set_passes(True)
        b.set_passes(True)
    assert status(lambda: binding._check(binding.load().lbm_set_passes(s.ctx, 2), "")) == binding.LBM_EINVAL
assert fake.fake_used() == 0
""")


def test_taking_a_second_buffer_breaks_no_capture(run):
    run("""
c = case((40, 36, 33))
with binding.Solver(c.params) as s:
    s.init(c.Q0)
    fake.fake_capture(0x777, 1)  # another stream's, in global mode
    s.step(9)
    fake.fake_capture(0x777, 0)
    assert s.passes()["second_bytes"] > 0 and not notes("BROKEN-CAPTURE")
""")


def test_second_buffers_go_to_allocations_from_any_thread(run):
    # one thread steps and reads out without a pause while the other's contexts need the
    # room: the buffer goes soon, after a wait for its owner's stream, and no step uses it
    # after that
    run("""
fake.fake_reset(520 << 20)
c, big = case((64, 64, 64)), case((96, 96, 96))
stop = threading.Event()
errors = []
with binding.Solver(c.params) as s:
    s.init(c.Q0)
    s.step(9)
    second = [value(n[3], "p") for n in notes("malloc") if value(n[3], "bytes") == s.passes()["second_bytes"]][-1]
    def work():
        try:
            while not stop.is_set():
                s.step(9)
                s.moments()
        except Exception as e:
            errors.append(e)
    t = threading.Thread(target=work)
    t.start()
    others = [binding.Solver(big.params) for _ in range(4)]  # 4 x 118 MiB beside 35 + 35
    stop.set()
    t.join()
    assert not errors and s.passes()["second_bytes"] == 0
    log = notes()
    assert len(log) < 50000
    freed = max(i for i, n in enumerate(log) if n[0] == "free" and value(n[3], "p") == second)
    stream = [n for n in log if n[0] == "launch"][0][1]
    waits = [i for i, n in enumerate(log) if n[0] == "sync" and n[1] == stream and n[2] == 0 and i < freed]
    assert waits
    last = max(waits)
    for n in log[last:]:
        assert n[0] != "launch" or second not in (value(n[3], "a0"), value(n[3], "a1"))
    for o in others:
        o.close()
assert fake.fake_used() == 0
""")


def test_pinned_user_memory_is_copied_directly(run):
    run("""
c = case((96, 64, 40))
lib, p = binding.load(), ctypes.c_void_p()
size = 35 * 4 * c.cells
fake.hipHostMalloc(ctypes.byref(p), ctypes.c_size_t(size), 0)
f, step = ctypes.cast(p, ctypes.POINTER(ctypes.c_float)), ctypes.c_int64()
q = ctypes.cast(p, ctypes.POINTER(ctypes.c_double))
with binding.Solver(c.params) as s:
    s.init(c.Q0)
    ctypes.memmove(p, np.ascontiguousarray(c.Q0).ctypes.data, 5 * 8 * c.cells)
    for call, n in ((lambda: lib.lbm_get_populations(s.ctx, f, ctypes.byref(step)), size),
                    (lambda: lib.lbm_set_populations(s.ctx, f, 0), size),
                    (lambda: lib.lbm_moments(s.ctx, q), 5 * 8 * c.cells)):
        fake.fake_reset(0)
        assert call() == 0
        (copy,) = notes("copy")
        assert value(copy[3], "bytes") == n and p.value in (value(copy[3], "dst"), value(copy[3], "src"))
""")


@pytest.mark.parametrize("dims,storage,least", [((256, 4, 4), "F16", 4), ((2000, 1, 1), "F16", 4),
                                                ((3000, 4, 4), "F16", 8), ((4097, 4, 4), "F16", 6),
                                                ((8192, 4, 4), "F16", 10),
                                                ((256, 4, 4), "F32", 4), ((4000, 5, 5), "F32", 6),
                                                ((20000, 4, 4), "F32", 6)])
def test_short_runs_of_tubes_are_single(run, dims, storage, least):
    run(f"""
c = case({dims})
with binding.Solver(c.params, storage={storage}) as s:
    s.init(c.Q0)
    for n in (1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12):
        s.step(s.step_count % 2)
        fake.fake_reset(0)
        s.step(n)
        passes = "k_step_tube" in kernels()
        assert passes == (n >= {least}), (n, kernels())
""")


def test_short_batch_runs_are_single(run):
    run("""
tubes = [((300, 4, 4), F32), ((300, 4, 4), F16)]
cubes = [((40, 36, 33), F32), ((24, 24, 24), F16)]
for insts, least in ((tubes, 4), (cubes, 8), (tubes + cubes, 8)):
    with binding.Batch(1 << 26, graph_steps=64) as b:
        for d, st in insts:
            c = case(d)
            b.add(c.params, c.Q0, 1000, storage=st)
        for n in (2, 4, 6, 8, 10):
            fake.fake_reset(0)
            b.run(n)
            fast = bool({"k_batch_pair", "k_batch_tube"} & set(kernels()))
            assert fast == (n >= least), (insts, n)
""")


@pytest.mark.parametrize("dims,cells", [((128, 128, 128), False), ((24, 24, 24), False), ((1, 64, 64), False),
                                        ((16, 512, 512), False), ((14, 512, 512), True),
                                        ((2 ** 31 - 1, 1, 1), True), ((1, 2 ** 31 - 1, 1), True),
                                        ((1, 1, 2 ** 31 - 1), True), ((2 ** 16, 2 ** 15, 1), False), ((2 ** 26, 2, 16), False),
                                        ((1, 2 ** 16, 2 ** 15), True)])
def test_source_kernel_of_a_lattice(run, dims, cells):
    # narrow ones are evaluated per cell; every size up to 2^31 cells can be launched, and
    # tiles are taken only where coordinates a tile past the end fit 32 bits
    run(f"""
dims, cells = {dims}, {cells}
m = inputs.mms(n=64).meta["mms"]
binding.lbm_mms_source(m, *dims, 0.5, 256)
assert kernels() == ["k_mms_source_cells" if cells else "k_mms_source"], kernels()
assert cells or max(dims) < 2 ** 31 - 64
""")


@pytest.mark.parametrize("storage", ["F32", "F16"])
@pytest.mark.parametrize("many,few,n", [((8000, 1, 1), (600, 5, 5), 12), ((3000, 4, 4), (1000, 5, 5), 12),
                                        ((1000, 5, 5), (9000, 2, 2), 12), ((1000, 5, 5), (3000, 4, 4), 6)])
def test_a_groups_windows_do_not_depend_on_the_order_of_its_tubes(run, many, few, n, storage):
    run(f"""
seen = []
for dims in ([{many}] * {n} + [{few}], [{few}] + [{many}] * {n}):
    with binding.Batch(1 << 29, graph_steps=64) as b:
        for d in dims:
            c = case(d)
            b.add(c.params, c.Q0, 1000, storage={storage})
        fake.fake_reset(0)
        b.run(30)
        seen.append([(value(n[3], "block"), value(n[3], "grid")) for n in notes("launch") if "k_batch_tube" in n[3]])
assert seen[0] and seen[0] == seen[1], seen
""")


def test_no_host_allocation_failure_leaves_a_call(run):
    # every operator new of a call fails in turn, and all after it: copies and checks go on
    # in the calling thread, a batch's run says so and can be made again
    run("""
c = case((96, 64, 40))
tubes = [case((300 + 50 * i, 4, 4)) for i in range(3)]
with binding.Solver(c.params) as s, binding.Batch(1 << 27, graph_steps=8) as b:
    f, Q = s.init(c.Q0) or (s.populations()[0], s.moments())
    ids = [b.add(t.params, t.Q0, 100) for t in tubes]
    b.run(8)
    calls = [(lambda: s.init(c.Q0), 0), (s.populations, 0), (s.moments, 0), (lambda: s.set_populations(f, 0), 0),
             (lambda: b.populations(ids[0]), 0), (lambda: b.run(9), binding.LBM_ENOMEM)]
    b.remove(ids.pop())
    for call, other in calls:
        for k in (range(6) if other == 0 else [0]):
            fail_new.fake_fail_new(k)
            st = status(call)
            fail_new.fake_fail_new(-1)
            assert st == other, (call, k, st)
    b.run(9)
    assert b.query(ids[0])[0] == 17
""")


def test_copies_without_pinned_slots(run):
    # none, fewer than the threads want, and one slot of two
    run("""
c = case((96, 64, 40))
for slots in (0, 1, 3, 16):
    fake.fake_slots(slots)
    with binding.Solver(c.params) as s:
        s.init(c.Q0)
        fake.fake_reset(0)
        f, _ = s.populations()
        q = s.moments()
        assert sum(value(n[3], "bytes") for n in notes("copy")) == (35 * 4 + 5 * 8) * c.cells
        # no kernel has run: both readouts hold what init left in the staging buffer
        assert np.array_equal(q, c.Q0) and np.array_equal(f.reshape(-1).view(np.float64)[:q.size], c.Q0.reshape(-1))
assert fake.fake_used() == 0
""")


def test_a_failed_allocation_is_reported_once(run):
    # the step after it, in another context, does not find its error
    run("""
fake.fake_reset(300 << 20)
c, big = case((40, 36, 33)), case((128, 128, 128))
with binding.Solver(c.params) as s, binding.Batch(1 << 26) as b:
    s.init(c.Q0)
    b.add(c.params, c.Q0, 100)
    for step in (lambda: s.step(9), lambda: b.run(9), lambda: s.step(1)):
        assert status(lambda: binding.Solver(big.params)) == binding.LBM_ENOMEM
        assert status(step) == 0
""")


@pytest.mark.parametrize("dims,storage", [((40, 36, 33), "F32"), ((300, 4, 4), "F16"), ((40, 36, 33), "F16")])
def test_passes_are_counted_as_launched(run, dims, storage):
    # what the benchmark divides its time and traffic by; also where no second buffer fits
    run(f"""
c = case({dims})
for room in (1 << 33, 40 << 20) if c.cells > 40000 else (1 << 33,):
    fake.fake_reset(room)
    with binding.Solver(c.params, storage={storage}) as s:
        big = binding.Solver(case((64, 64, 57)).params) if room < 1 << 33 else None  # 33 MB: the card is full
        s.init(c.Q0)
        for n, every in ((1, 0), (2, 0), (15, 0), (40, 7), (40, 20), (9, 1), (33, 3), (64, 0), (50, 50)):
            before = s.passes()
            fake.fake_reset(0)
            s.step(n, every)
            after = s.passes()
            steps = [k for k in kernels() if k.startswith("k_step")]
            assert after["steps"] - before["steps"] == n
            assert after["passes"] - before["passes"] == len(steps), (n, every, steps)
            assert not big or (after["second_bytes"] == 0 and len(steps) == n)
        if big:
            big.close()
""")


def test_the_second_arena_is_as_large_as_its_instances_need(run):
    run("""
small, large, plain = case((300, 4, 4)), case((60, 60, 60)), case((64, 64, 64))
with binding.Batch(1 << 29, graph_steps=8) as b:
    def held():
        return b.passes()["second_bytes"] >> 20
    for _ in range(3):
        b.add(plain.params, plain.Q0, 1000, storage=F16)  # 18 MB each, in single steps
    b.run(8)
    assert held() == 0
    b.add(small.params, small.Q0, 1000)
    assert held() == 64
    b.run(8)
    assert held() == 64
    ids = [b.add(large.params, large.Q0, 1000) for _ in range(4)]  # 30 MB each
    fake.fake_reset(0)
    b.run(16)
    assert held() == 256 and b.passes()["fast_steps"] == 24
    log = notes()
    freed = [i for i, n in enumerate(log) if n[0] == "free"]
    assert len(freed) == 1 and any(n[0] == "sync" for n in log[:freed[0]])
    assert any(n[0] == "destroy-graph" for n in log)  # the one that names the old arena
    seconds = {x for n in notes("launch") for x in (value(n[3], "a0"), value(n[3], "a1")) if "k_batch_pair" in n[3]}
    gone = value(log[freed[0]][3], "p")
    assert len(seconds) == 2 and gone not in seconds
    for i in ids:
        b.remove(i)
    b.run(8)
    assert held() == 256  # kept
assert fake.fake_used() == 0
""")


def test_short_solves_in_new_contexts_take_no_second_buffer(run):
    run("""
for dims, steps, takes in (((64, 64, 64), 40, False), ((64, 64, 64), 70, True), ((128, 128, 64), 16, True),
                           ((40, 36, 33), 4, True)):
    c = case(dims)
    for parts in ((steps,), (steps // 2, steps - steps // 2)):
        with binding.Solver(c.params) as s:
            binding.lbm_init_fields_device(s.ctx, np.ascontiguousarray(c.Q0).ctypes.data)
            for n in parts:
                s.step(n)
            assert (s.passes()["second_bytes"] > 0) == takes or parts[-1] < 3, (dims, parts)
""")


def test_a_batchs_clock_is_the_devices_where_a_run_fails(run):
    # a graph of eight steps is on its way when the rest of the run fails: they count
    run("""
c = case((24, 24, 24))
for storage, after, done, kept in ((F16, 0, 16, True), (F16, 3, 16, False)):
    with binding.Batch(1 << 26, graph_steps=8) as b:
        i = b.add(c.params, c.Q0, 1000, storage=storage)
        b.run(8)
        fake.fake_fail(b"k_batch_step", after)
        assert status(lambda: b.run(13)) == binding.LBM_EDEVICE
        assert b.query(i)[0] == done and b.info()["clock"] == done
        assert status(lambda: b.run(1)) == (0 if kept else binding.LBM_ESTATE)
""")


def test_instances_that_finish_before_a_failure_are_listed_no_more(run):
    run("""
c, d = case((24, 24, 24)), case((30, 30, 30))
with binding.Batch(1 << 26, graph_steps=8) as b:
    i, j = b.add(c.params, c.Q0, 16, storage=F16), b.add(d.params, d.Q0, 1000, storage=F16)
    b.run(8)
    fake.fake_fail(b"k_batch_step", 0)
    assert status(lambda: b.run(13)) == binding.LBM_EDEVICE
    assert b.query(i) == (16, True) and b.query(j) == (16, False)
    fake.fake_reset(0)
    b.run(8)
    assert notes("copy")  # the lists, without the finished one
    assert b.query(j)[0] == 24
""")


def test_batches_of_single_steps_hold_one_tile_list(run):
    run("""
fp16, fp32 = case((24, 24, 24)), case((40, 36, 33))
for room in (1 << 33, 130 << 20):  # the second list of 100 MB does not fit beside the first
    fake.fake_reset(room)
    with binding.Batch(1 << 22, max_tiles=3 << 20) as b:
        own = fake.fake_used()
        assert own < 110 << 20
        b.add(fp16.params, fp16.Q0, 1000, storage=F16)
        b.run(8)
        assert fake.fake_used() == own
    with binding.Batch(1 << 23, max_tiles=3 << 20) as b:
        b.add(fp32.params, fp32.Q0, 1000)
        b.run(32)
        assert b.passes()["fast_steps"] == (32 if room > 1 << 30 else 0)
assert fake.fake_used() == 0
""")


def test_a_second_buffer_is_taken_once_and_on_its_own_device(run):
    run("""
c = case((40, 36, 33))
with binding.Solver(c.params) as s, binding.Batch(1 << 26) as b:
    s.init(c.Q0)
    b.add(c.params, c.Q0, 1000)
    s.step(9)
    b.run(16)
    own = fake.fake_used()
    for _ in range(2):
        s.set_passes(True)  # it is on already
        b.set_passes(True)
        s.step(9)
        b.run(16)
        assert fake.fake_used() == own
    s.set_passes(False)
    b.set_passes(False)
    less = fake.fake_used()
    s.set_passes(True)
    b.set_passes(True)
    fake.hipSetDevice(1)  # the caller's other device
    s.step(9)
    b.run(16)
    assert fake.fake_used() == less
    fake.hipSetDevice(0)
    s.step(9)
    b.run(16)
    assert fake.fake_used() == own
assert fake.fake_used() == 0
""")
