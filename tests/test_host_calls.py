"""The library's host side on the CPU, against a stand-in for the HIP runtime
(tests/host/mock_hip.cpp, loaded ahead of it in a child process): which runtime
calls an entry point makes, and what it does when one fails."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2601_01903_amd", "_lib", "libfsi_mi355x.so")

PRELUDE = r"""
import ctypes as C
mock = C.CDLL({mock!r}, mode=C.RTLD_GLOBAL)   # its symbols come first
mock.mock_log.restype = C.c_char_p
mock.mock_fail_malloc.argtypes = [C.c_size_t, C.c_int]
lib = C.CDLL({lib!r})
lib.fsi_last_error.restype = C.c_char_p
vp, i32 = C.c_void_p, C.c_int
for name in ("fsi_apply", "fsi_apply_batched", "fsi_apply_batched_nograph"):
    getattr(lib, name).argtypes = [vp] * 4
lib.fsi_forest_values.argtypes = [vp, vp, i32, vp, i32, vp, vp]
for name in ("fsi_plan_destroy", "fsi_batch_plan_destroy", "fsi_forest_destroy"):
    getattr(lib, name).argtypes = [vp]
def log():
    return mock.mock_log().decode().splitlines()
def launches():   # (grid, dynamic LDS bytes, kernel)
    return [(int(g), int(b), k) for g, b, k in (x.split(" ", 3)[1:] for x in log() if x.startswith("launch"))]
def ok(status):
    assert status == 0, lib.fsi_last_error()
def stream():
    s = vp()
    ok(mock.hipStreamCreateWithFlags(C.byref(s), 1))
    return s
def ints(x):
    return (i32 * len(x))(*x)
def batch(ds, ls, opts=None):
    p = vp()
    ok(lib.fsi_plan_batched(len(ds), ints(ds), ints(ls), opts, C.byref(p)))
    return p
buf = C.create_string_buffer((1 << 20) + 64)
A = (C.addressof(buf) + 63) & ~63
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("mock") / "libmock_hip.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", "-Wno-unused-result",
                    os.path.join(ROOT, "tests", "host", "mock_hip.cpp"), "-o", so], check=True)

    def go(code, **env):
        src = PRELUDE.format(mock=so, lib=LIB) + code + "\nprint('done')\n"
        r = subprocess.run([sys.executable, "-c", src], capture_output=True, text=True, timeout=120,
                           env=dict(os.environ, **dict({"FSI_TUNE_CACHE": ""}, **env)))
        assert r.returncode == 0 and r.stdout.strip().endswith("done"), r.stdout + r.stderr
        return r.stdout
    return go


def test_destroy_after_the_stream(run):
    """A plan outlives the streams it ran on: destroying it names none of them,
    and the memory is freed (which waits for the device) before the graph."""
    run(r"""
for call in ("fsi_apply_batched", "fsi_apply_batched_nograph"):
    p, s = batch([12, 9], [3, 2]), stream()
    ok(getattr(lib, call)(p, A, A, s))
    ok(mock.hipStreamDestroy(s))
    log()
    ok(lib.fsi_batch_plan_destroy(p))
    calls = log()
    assert not [x for x in calls if x.startswith("DEAD_STREAM")], calls
    names = [x.split()[0] for x in calls]
    if call == "fsi_apply_batched":
        assert names.index("hipFree") < names.index("hipGraphExecDestroy"), calls
    assert "hipFree" in names
""")


def test_small_launches_leave_room(run):
    """A launch of at most one workgroup per CU asks for its own LDS only, so that
    another stream's fits beside it on the CU's 160 KB."""
    run(r"""
for d, l, n in [(14, 3, 1), (20, 4, 1), (11, 1, 250), (14, 3, 30)]:
    opts = (i32 * 10)()
    ok(lib.fsi_default_opts(opts))
    opts[0] = 1                       # FP32 storage
    p = batch([d] * n, [l] * n, opts)
    log()
    ok(lib.fsi_apply_batched_nograph(p, A, A, None))
    tile = [x for x in launches() if "tile11" in x[2]]
    assert len(tile) == 1 and tile[0][0] <= 256 and 2 * tile[0][1] <= 160 * 1024, (d, l, n, tile)
    ok(lib.fsi_batch_plan_destroy(p))
""")


def test_tune_entries_of_other_schedules(run, tmp_path):
    """An entry written when the same numbers meant another schedule (its key has
    no schedule version) is not taken: the plan is timed, and its own entry serves
    the next process."""
    path = tmp_path / "tune.json"
    code = r"""
import struct
opts = (i32 * 10)()
ok(lib.fsi_default_opts(opts))
opts[5] = 1                       # autotune
key = "gfx950-256cu/%d/%d/%d/%d/%d/%d;12,6x1" % tuple(opts[i] for i in (0, 1, 2, 6, 3, 8))
p = batch([12], [6], opts)
s = C.create_string_buffer(24)
ok(lib.fsi_batch_schedule(p, s))
print("KEY", key)
print("SCHED", *struct.unpack("5if", s.raw))
ok(lib.fsi_batch_plan_destroy(p))
"""
    def sched(out):
        return [x.split()[1:] for x in out.splitlines() if x.startswith("SCHED")][0]
    out = run(code, FSI_TUNE_CACHE=str(tmp_path / "other.json"))
    key = [x[4:] for x in out.splitlines() if x.startswith("KEY")][0]
    path.write_text('{"format": "fsi-autotune-1", "entries": [\n{"key": "%s", "kernel": 1, "tb_shift": '
                    '-2, "chunk_shift": 0, "mob_group": 0, "algo": 1}\n]}\n' % key)
    first = sched(run(code, FSI_TUNE_CACHE=str(path)))
    assert first[0] == "1" and first[3] == "0" and float(first[5]) > 0
    second = sched(run(code, FSI_TUNE_CACHE=str(path)))
    assert second[0] == "1" and second[3] == "0" and float(second[5]) == 0


def test_forest_without_room_for_its_lists(run):
    """The leaf lists of the walk are optional: a forest whose device has no room
    for them is made all the same, and its walk runs without the listing pass."""
    run(r"""
import math
d, trees, bgs = 16, 40, 200
D, F64 = C.c_double, C.c_double * (3 * trees)
f, l, r = ints([0, -1, -1] * trees), ints([3 * k + 1 for k in range(trees) for _ in range(3)]), ints([3 * k + 2 for k in range(trees) for _ in range(3)])
z = F64()
def values(fail):
    h = vp()
    mock.mock_fail_malloc(1 << 20, fail)
    ok(lib.fsi_forest_create(d, trees, ints(range(0, 3 * trees, 3)), 3 * trees, f, z, l, r, z, bgs, C.byref(h)))
    mock.mock_fail_malloc(0, 0)
    log()
    ok(lib.fsi_forest_values(h, A, bgs, A, 0, A, None))
    names = [k for _, _, k in launches()]
    ok(lib.fsi_forest_destroy(h))
    return names
assert any("reach" in k for k in values(0))
names = values(1)
assert not any("reach" in k for k in names) and any("walk" in k for k in names), names
""")


def test_plans_at_the_scratch_line_are_built_once(run):
    """Orders 5 and 6 keep the generic kernel where only its results fit the scratch
    of the call without allocation: making such a plan takes the time of a
    generic one."""
    run(r"""
import time
for d, l, n in [(18, 5, 24), (20, 5, 7)]:
    best = [1e9, 1e9]
    for _ in range(9):
        for kernel in (0, 1):
            opts = (i32 * 10)()
            ok(lib.fsi_default_opts(opts))
            opts[0], opts[6] = 1, kernel
            t = time.perf_counter()
            p = batch([d] * n, [l] * n, opts)
            best[kernel] = min(best[kernel], time.perf_counter() - t)
            log()
            ok(lib.fsi_apply_batched_nograph(p, A, A, None))
            assert not any("tile_high" in k for _, _, k in launches())
            ok(lib.fsi_batch_plan_destroy(p))
    assert best[0] < 1.8 * best[1], (d, l, n, best)
""")


def test_result_counts_of_the_generic_kernel(tmp_path):
    csrc = os.path.join(ROOT, "paper_2601_01903_amd", "csrc")
    exe = str(tmp_path / "check")
    subprocess.run(["hipcc", "-O1", "-std=c++17", "-I" + os.path.join(ROOT, "include"), "-I" + csrc,
                    os.path.join(ROOT, "tests", "host", "check_tile_results.cpp"),
                    os.path.join(csrc, "fsi_tables.cpp"), "-o", exe], check=True, capture_output=True)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out.stdout
