"""Which kernels the library's host side launches, without a GPU: libqaia in a
process of its own on a HIP runtime of host memory (fake_hip.cpp), which notes
the launches by name."""
import os
import subprocess
import sys
import textwrap

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PRELUDE = """
import ctypes as C
import sys
import numpy as np
fake = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
lib = C.CDLL(sys.argv[2])
fake.fake_limit.argtypes = [C.c_size_t]
fake.fake_in_use.restype = C.c_size_t
lib.qaia_last_error.restype = C.c_char_p


class Schedule(C.Structure):
    _fields_ = [("variant", C.c_int32), ("precision", C.c_int32), ("steps", C.c_int32), ("path", C.c_int32),
                ("dt", C.c_float), ("a0", C.c_float), ("init_amp", C.c_float), ("noise_alpha", C.c_float),
                ("seed", C.c_uint64), ("replica_offset", C.c_uint64)]


class Item(C.Structure):
    _fields_ = [("problem", C.c_void_p), ("weights", C.c_void_p), ("W", C.c_int64), ("R", C.c_int32),
                ("path", C.c_int32), ("spins", C.c_void_p), ("obj", C.c_void_p), ("tile", C.c_int32),
                ("reserved", C.c_int32)]


def ok(rc):
    assert rc == 0, (rc, lib.qaia_last_error())


def ptr(a):
    return a.ctypes.data_as(C.c_void_p)


def count(name):
    return fake.fake_count(name.encode())


def edges(n, density, seed=1):
    u, v = np.triu_indices(n, 1)
    keep = np.random.default_rng(seed).random(u.size) < density
    return u[keep].astype(np.int32), v[keep].astype(np.int32)


def ring(n):
    u = np.arange(n - 1, dtype=np.int32)
    return u, u + 1


def problem(n, m, u, v, largest):
    w = np.random.default_rng(n).integers(-largest, largest + 1, size=(m, u.size)).astype(np.int32)
    p = C.c_void_p()
    ok(lib.qaia_problem_create(n, m, C.c_int64(u.size), ptr(u), ptr(v), ptr(w), 16, 0, C.byref(p)))
    return p


def buffers(n, m, rows):
    return np.zeros((rows, (n + 63) // 64), np.int64), np.zeros((rows, m), np.int64)


def sample(p, n, m, W, R, s):
    c, (spins, obj), need = np.full((W, m), 1.0 / m, np.float32), buffers(n, m, W * R), C.c_size_t()
    ok(lib.qaia_sample_workspace_bytes(p, C.c_int64(W), R, C.byref(s), C.byref(need)))
    ws = np.zeros(need.value, np.uint8)
    fake.fake_clear()
    ok(lib.qaia_sample(p, ptr(c), C.c_int64(W), R, C.byref(s), ptr(spins), ptr(obj), ptr(ws), need, None))


def batch(items, s):
    # items: (problem, n, m, W, R)
    keep, arr = [], (Item * len(items))()
    for a, (p, n, m, W, R) in zip(arr, items):
        c, (spins, obj) = np.full((W, m), 1.0 / m, np.float32), buffers(n, m, W * R)
        keep += [c, spins, obj]
        a.problem, a.weights, a.W, a.R, a.path = p, c.ctypes.data, W, R, 4
        a.spins, a.obj = spins.ctypes.data, obj.ctypes.data
    need = C.c_size_t()
    ok(lib.qaia_sample_batch_workspace_bytes(arr, len(items), C.byref(s), C.byref(need)))
    ws = np.zeros(need.value, np.uint8)
    fake.fake_clear()
    ok(lib.qaia_sample_batch(arr, len(items), C.byref(s), ptr(ws), need, None))


BSB, DSB, FP32, BF16, FP8 = 0, 1, 0, 1, 2
AUTO, SPARSE_REG, SPARSE_LDS, DENSE, STAGED = range(5)
SMALL, LARGE = 1000, 1 << 22  # weights whose rows stay below 2^24 (exact digits), and not
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    lib = os.path.join(ROOT, "paper_2604_26477_amd", "libqaia.so")
    so = str(tmp_path_factory.mktemp("fake") / "libfakehip.so")
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-std=c++17", "-o", so, os.path.join(ROOT, "tests", "fake_hip.cpp")],
                   check=True)

    def go(body, *args, jit=False):
        env = {k: v for k, v in os.environ.items() if k != "QAIA_DISABLE_JIT"}
        if not jit:
            env["QAIA_DISABLE_JIT"] = "1"
        r = subprocess.run([sys.executable, "-c", PRELUDE + textwrap.dedent(body), so, lib, *map(str, args)],
                           capture_output=True, text=True, env=env, timeout=300)
        assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]
    return go


# ---------------------------------------------------------------- batch

@pytest.mark.parametrize("n,items,W,R,variant,precision,largest,grouped", [
    (300, 30, 8, 8, "BSB", "FP32", "LARGE", True),   # many, few columns: one grouped launch per step
    (512, 48, 32, 32, "BSB", "FP32", "LARGE", True),
    (512, 24, 8, 8, "DSB", "BF16", "LARGE", True),
    (512, 3, 8, 8, "BSB", "FP32", "LARGE", False),   # as many as there are branches
    (300, 1, 8, 8, "BSB", "FP32", "LARGE", False),
    (400, 24, 64, 64, "BSB", "FP32", "LARGE", False),  # each fills much of the chip
    (70, 48, 8, 8, "DSB", "FP32", "SMALL", False),   # exact digits
])
def test_batch_of_staged_items_takes_the_shorter_way(run, n, items, W, R, variant, precision, largest, grouped):
    """Staged items of up to 512 spins are a launch each only where that is the
    shorter way; never a launch per item and step (the thin tiles of single calls)."""
    run("""
    n, k, W, R, grouped = (int(x) for x in sys.argv[3:8])
    m, T = 2, 40
    s = Schedule(%s, %s, T, AUTO, 0.5, 1.0, 0.1, 0.0, 1, 0)
    p = problem(n, m, *edges(n, 0.3), %s)
    batch([(p, n, m, W, R)] * k, s)
    one = count("resident_kernel") + count("digits_kernel")
    steps = count("dense_batch_step_staged")
    assert count("dense_thin") == 0 and count("dense_step") == 0
    assert (one, steps) == ((0, T) if grouped else (k, 0)), (one, steps)
    """ % (variant, precision, largest), n, items, W, R, int(grouped))


def test_batch_of_small_and_large_staged_items(run):
    """Items past 512 spins stay in the grouped steps, whatever the others take."""
    run("""
    s = Schedule(BSB, FP32, 20, AUTO, 0.5, 1.0, 0.1, 0.0, 1, 0)
    big, small = problem(600, 3, *edges(600, 0.1), LARGE), problem(64, 3, *edges(64, 0.5), LARGE)
    batch([(big, 600, 3, 8, 8), (small, 64, 3, 8, 8), (small, 64, 3, 0, 8)], s)
    assert count("dense_batch_step_staged") == 20 and count("resident_kernel") == 1
    """)


# ---------------------------------------------------------------- single calls

def test_few_replicas_leave_the_generated_kernel_only_for_runs_long_enough(run):
    """AUTO on a graph of the generated kernel: one spin per lane for few replicas
    and enough steps for its set-up and read-out, both sides of each line."""
    run("""
    cases = [  # n, complete, m, rows, steps, noise, one spin per lane
        (12, 0, 3, 256, 55, 0.0, 0), (12, 0, 3, 256, 56, 0.0, 1), (12, 0, 3, 4096, 200, 0.0, 1), (12, 0, 3, 4097, 200, 0.0, 0),
        (2, 0, 3, 64, 1000, 0.0, 0), (42, 0, 4, 1, 4, 0.0, 0), (42, 0, 4, 1, 5, 0.0, 1), (42, 0, 4, 16384, 65, 0.0, 0),
        (42, 0, 4, 16384, 66, 0.0, 1), (42, 0, 4, 16385, 1000, 0.0, 0), (42, 0, 5, 1, 7, 0.0, 0), (42, 0, 5, 1, 8, 0.0, 1),
        (16, 1, 3, 64, 15, 0.0, 0), (16, 1, 3, 64, 16, 0.0, 1), (16, 1, 3, 6400, 21, 0.0, 0), (16, 1, 3, 6400, 22, 0.0, 1),
        (16, 1, 3, 6401, 1000, 0.0, 0), (14, 1, 3, 1, 1000, 0.0, 0),
        (12, 0, 3, 64, 6, 0.2, 0), (12, 0, 3, 64, 7, 0.2, 1), (12, 0, 3, 40000, 26, 0.2, 0), (12, 0, 3, 40000, 27, 0.2, 1),
        (12, 0, 3, 40001, 1000, 0.2, 0), (16, 1, 3, 25000, 24, 0.2, 0), (16, 1, 3, 25000, 25, 0.2, 1)]
    made = {}
    for n, complete, m, rows, steps, noise, group in cases:
        key = n, complete, m
        if key not in made:
            made[key] = problem(n, m, *(edges(n, 1.1) if complete else ring(n)), SMALL)
        sample(made[key], n, m, rows, 1, Schedule(BSB, FP32, steps, AUTO, 1.0, 1.0, 0.1, noise, 1, 0))
        assert (count("group_kernel"), count("generated")) == (group, 1 - group), (n, m, rows, steps, noise)
    """, jit=True)


# ---------------------------------------------------------------- problems

@pytest.mark.parametrize("n,degree,order", [(1024, 2, True), (1025, 2, False), (200, 33, False)])
def test_only_graphs_of_the_one_spin_per_lane_kernel_get_its_lane_order(run, n, degree, order):
    """The device memory of a graph without images: its edges, weights, lists and row
    sums, and the order of that kernel (up to 1024 nodes and degree 32) where it runs."""
    run("""
    n, degree, order = (int(x) for x in sys.argv[3:6])
    m = 8
    u, v = ring(n)
    if degree > 2:
        u, v = np.concatenate([u, np.zeros(degree - 1, np.int32)]), np.concatenate([v, np.arange(2, degree + 1, dtype=np.int32)])
    E = u.size
    p = problem(n, m, u, v, SMALL)
    plain = 4 * (2 * E + m * E + (n + 1) + 4 * E) + 8 * m * n
    assert fake.fake_in_use() - plain == (8 * n if order else 0), (fake.fake_in_use(), plain)
    ok(lib.qaia_problem_destroy(p))
    assert fake.fake_in_use() == 0
    """, n, degree, int(order))


def test_problem_without_room_for_the_images_of_small_dense_graphs(run):
    """The fragment and digit images only make calls faster: where their allocation
    fails, the problem is created without them and the step kernels run."""
    run("""
    n, m = 512, 3
    fake.fake_limit(4 << 20)  # the dense images take 3 MiB, their fragments and digits 8
    for largest, variant in ((LARGE, BSB), (SMALL, DSB)):
        p = problem(n, m, *edges(n, 1.1), largest)
        assert fake.fake_sticky() == 0
        sample(p, n, m, 64, 64, Schedule(variant, FP32, 7, STAGED, 0.5, 1.0, 0.1, 0.0, 1, 0))
        assert count("dense_step_staged") + count("dense_thin") == 7
        assert count("resident_kernel") + count("digits_kernel") == 0
        batch([(p, n, m, 8, 8)] * 2, Schedule(variant, FP32, 7, AUTO, 0.5, 1.0, 0.1, 0.0, 1, 0))
        assert count("dense_batch_step_staged") == 7 and count("resident_kernel") + count("digits_kernel") == 0
        ok(lib.qaia_problem_destroy(p))
    assert fake.fake_in_use() == 0
    """)


def test_problem_without_room_for_the_cut_images(run):
    """Nor does a problem need the digit matrices of the cuts: the edges are walked."""
    run("""
    n, m = 512, 8
    fake.fake_limit(5 << 20)  # the weights take 4 MiB, the matrices 6
    p = problem(n, m, *edges(n, 1.1), LARGE)
    assert fake.fake_sticky() == 0
    spins, obj = buffers(n, m, 100)
    fake.fake_clear()
    ok(lib.qaia_evaluate(p, ptr(spins), C.c_int64(100), ptr(obj), None))
    assert count("eval_tile_kernel") == 1 and count("cut_kernel") == 0
    ok(lib.qaia_problem_destroy(p))
    assert fake.fake_in_use() == 0
    fake.fake_limit(3 << 20)  # the weights themselves do not fit
    w = np.ones((m, edges(n, 1.1)[0].size), np.int32)
    u, v = edges(n, 1.1)
    rc = lib.qaia_problem_create(n, m, C.c_int64(u.size), ptr(u), ptr(v), ptr(w), 16, 0, C.byref(C.c_void_p()))
    assert rc == 3 and fake.fake_in_use() == 0
    """)


# ---------------------------------------------------------------- cuts

@pytest.mark.parametrize("n,extra,m,count,walk", [(73, 12, 8, 570_000, True), (73, 12, 8, 100_000, False), (65, 10, 4, 570_000, True),
                                                  (65, 10, 4, 1000, False), (64, 10, 4, 570_000, False), (73, 300, 8, 570_000, False)])
def test_cuts_of_few_edges_and_many_samples_walk_the_edges(run, n, extra, m, count, walk):
    """Graphs with cut images still walk their edges where many samples make that shorter."""
    run("""
    n, extra, m, samples, walk = (int(x) for x in sys.argv[3:8])
    u, v = ring(n)
    a, b = np.triu_indices(n, 2)
    u, v = np.concatenate([u, a[:extra].astype(np.int32)]), np.concatenate([v, b[:extra].astype(np.int32)])
    p = problem(n, m, u, v, LARGE)
    spins, obj = buffers(n, m, samples)
    fake.fake_clear()
    ok(lib.qaia_evaluate(p, ptr(spins), C.c_int64(samples), ptr(obj), None))
    assert (count("eval_thread_kernel"), count("cut_kernel")) == (walk, 1 - walk)
    """, n, extra, m, count, int(walk))


def test_every_one_spin_per_lane_kernel_is_reached(run):
    """No instance is built that no call launches: spins, degrees, replicas, noise
    and variants on both sides of every rule of the choice."""
    run("""
    fake.fake_kernels.restype = C.c_char_p
    names = lambda launched: {k for k in fake.fake_kernels(launched).decode().split() if "group_kernel" in k}
    built, seen = names(0), set()
    for n in (20, 40, 100, 200, 400, 700):
        m = 8 if n == 20 else 1  # few edges per replica and objective: the read-out of several groups in a wave
        for degree in (2, 6, 19):
            u, v = ring(n)
            if degree > 2:
                u, v = np.concatenate([u, np.zeros(degree - 1, np.int32)]), np.concatenate([v, np.arange(2, degree + 1, dtype=np.int32)])
            p = problem(n, m, u, v, SMALL)
            for lanes in (1 << 17, 600_000, 700_000, 1_500_000):
                for R in (3, lanes // n):
                    for variant in (BSB, DSB):
                        for noise in (0.0, 0.1):
                            s = Schedule(variant, FP32, 3, SPARSE_LDS, 0.5, 1.0, 0.1, noise, 1, 0)
                            sample(p, n, m, -(-lanes // n // R), R, s)
                            seen |= names(1)
    assert built and seen == built, sorted(built - seen)
    """)
