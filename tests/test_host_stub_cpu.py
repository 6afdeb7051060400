"""The library's host code on the CPU: liboct on a HIP runtime without a device
(tests/sanitize/hip_stub.c), whose launches leave the kernels' names.  Which
kernels a plan's calls take, and every entry point under the host sanitizers."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
STUB = os.path.join(HERE, "sanitize", "hip_stub.c")
LIB = os.path.join(os.path.dirname(HERE), "paper_2108_01438_amd", "liboct.so")
DRIVER = os.path.join(HERE, "sanitize", "host_sanitize_driver")


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    d = tmp_path_factory.mktemp("hip_stub")
    out = os.path.join(d, "libamdhip64.so.7")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-Wl,-soname,libamdhip64.so.7", STUB, "-o", out], check=True)
    return out


# A process of its own: this one may hold the real runtime under the same name.
CHILD = r"""
import ctypes, math, struct, sys
stub = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
stub.stub_log.restype = ctypes.c_char_p
P = ctypes.c_void_p
BUF = P(4096)
BUF8 = ctypes.byref(ctypes.c_double())

def plan(n_depth, n_x, n_k, n_y=1, lateral_dims=1, kb_width=6, batch=1, k_min=2 * math.pi / 0.9, k_max=2 * math.pi / 0.75,
         dz=0.0, masked=False):
    g = struct.pack("<ii5q11dii", lateral_dims, kb_width, n_depth, n_x, n_y, n_k, batch, k_min, k_max, 2.0, 2.0, dz, -1.0,
                    5.0, 1e-3, 0.0, 2.0, 0.0, 0, 0)
    mask = (b"\1\0" * (n_x * n_y * n_k))[:n_x * n_y * n_k] if masked else None
    h = P()
    st = lib.oct_plan_create(ctypes.c_char_p(g), ctypes.c_char_p(mask), ctypes.byref(h))
    assert st == 0, (st, n_depth)
    return h

def kernels(f, *args):
    stub.stub_log_clear()
    st = f(*args)
    return st, [l.split()[0] for l in stub.stub_log().decode().splitlines()]

def columns(names):
    return [n for n in names if "column_pair" in n or "nufft" in n]
"""


def run_child(stub, code):
    r = subprocess.run([sys.executable, "-c", CHILD + code, stub, LIB], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-3000:]
    return r.stdout


def test_columns_by_grid_cell_only_with_distinct_cells(stub):
    """Samples are found by grid cell only where rounding cannot put two of them into one: not where
    the q = 0 coordinates k_min / dk + m lie within 2^-13 below an integer."""
    out = run_child(stub, r"""
eps = 2.0 ** -13
for n, t0, h, cell in [
    (512, 2560.0, 1.0, True), (512, 2560.0 - 1e-9, 1.0, True), (512, 2560.5, 1.0, True), (512, 2561.0 - 2 * eps, 1.0, True),
    (512, 2561.0 - eps, 1.0, False), (1024, 20001.0 - eps + 1e-11, 1.0, False), (512, 2561.0 - eps - 1e-8, 1.0, False),
    (2048, 9000.0 - 0.5 * eps, 1.0, False), (512, 2561.0 - 2e-5, 1.0, False),
    # half a cell more per sample than one, or a band over which the fraction runs into the boundary
    (512, 2561.0 - eps, 1.5, True), (512, 2561.0 - eps - 2e-6, 1.0 + 5e-9, False), (512, 2561.0 - 3e-4, 0.999, False),
]:
    dk = 1.4 / n                       # t = K dz / pi (k_min + m dk): h cells a sample
    h_plan = plan(n, 6, n - 1, k_min=t0 * dk / h, k_max=(t0 / h + n - 2) * dk, dz=h * math.pi / (2 * n * dk) if h != 1 else 0.0)
    for f, args in ((lib.oct_forward, (BUF, BUF, None)), (lib.oct_adjoint, (BUF, BUF, None)), (lib.oct_grad, (BUF, BUF, BUF, None, None))):
        st, names = kernels(f, h_plan, *args)
        got = columns(names)
        assert st == 0 and got and all(("column_pair" in k) == cell for k in got), (n, t0, h, cell, got)
print("ok")
""")
    assert out.strip() == "ok"


def test_stages_run_the_kernels_of_the_calls(stub):
    """oct_run_stage launches what oct_forward, oct_adjoint and oct_grad launch, fully observed or
    masked, where the columns run by grid cell (1225: its K-point rows fit no pair kernel) and where
    they do not (2000)."""
    out = run_child(stub, r"""
for n in (512, 1225, 1400, 2000):
    for masked in (False, True):
        p = plan(n, 4, n, masked=masked)
        cell = n != 2000
        def stage(k):
            st, names = kernels(lib.oct_run_stage, p, k, 0, BUF, None)
            assert st == 0
            return columns(names)
        fwd, adj = columns(kernels(lib.oct_forward, p, BUF, BUF, None)[1]), columns(kernels(lib.oct_adjoint, p, BUF, BUF, None)[1])
        both = columns(kernels(lib.oct_lipschitz, p, 1, ctypes.c_uint64(0), 0, BUF8, None)[1])
        assert len(fwd) == len(adj) == 1 and len(both) == (2 if masked else 1)
        assert all(("column_pair" in k) == cell for k in fwd + adj + both), (n, fwd, adj, both)
        assert stage(3) == adj
        if masked or cell:
            assert stage(1) == fwd, (n, masked, stage(1), fwd)
        else:
            assert len(stage(1)) == 1
        if not masked:
            assert stage(6) == both
print("ok")
""")
    assert out.strip() == "ok"


def test_small_and_narrow_volumes_step_in_two_kernels(stub):
    """3-D TV: the walk along y where a volume fills its tiles, two kernels per step where it is
    small or a few rows wide; a few steps on a small one are one pass of the walk."""
    out = run_child(stub, r"""
def prox(nz, nx, ny, inner, batch=1):
    p = plan(nz, nx, nz, n_y=ny, lateral_dims=2, batch=batch)
    f = lib.oct_prox
    D = ctypes.c_double
    st, names = kernels(f, p, 1, D(0.1), D(1.0), inner, 1, D(0.0), BUF, P(8192), None, None)
    assert st == 0
    lib.oct_plan_destroy(p)
    return sum("tv3d_march" in n for n in names), sum("tv_step" in n for n in names)
for args, walks in [((128, 16, 16, 10), False), ((2048, 8, 8, 10), False), ((1024, 4, 100, 10), False), ((1024, 1, 256, 20), False),
                    ((256, 40, 45, 10), True), ((512, 32, 32, 10), True), ((512, 64, 64, 20), True), ((1024, 96, 96, 10), True),
                    ((128, 16, 16, 3), False), ((128, 16, 16, 2), True), ((1024, 96, 96, 1), True)]:
    march, step = prox(*args)
    n = args[3]
    assert (march, step) == ((-(-n // 3), 0) if walks else (0, n)), (args, march, step)
print("ok")
""")
    assert out.strip() == "ok"


# checks of values that kernels compute, which do nothing here
VALUES = {"lipschitz positive", "ncc", "nothing observed: the solution is exactly zero"}


def test_every_entry_point_under_host_sanitizers(stub):
    """tests/sanitize/host_sanitize_driver.cpp with AddressSanitizer, UndefinedBehaviorSanitizer and
    the leak check on the library's host code: no report, and every status as declared."""
    assert os.path.exists(DRIVER), f"{DRIVER} is missing: run __graft_entry__.build()"
    env = dict(os.environ, LD_LIBRARY_PATH=os.path.dirname(stub), ASAN_OPTIONS="halt_on_error=1:detect_leaks=1:exitcode=99",
               LSAN_OPTIONS="exitcode=98", UBSAN_OPTIONS="halt_on_error=1:print_stacktrace=1")
    r = subprocess.run([DRIVER], capture_output=True, text=True, timeout=120, env=env)
    bad = {l.split(": ", 1)[1].split(" (last error")[0] for l in r.stderr.splitlines() if l.startswith("UNEXPECTED")}
    assert r.returncode in (0, 1) and "335 checks" in r.stderr, (r.returncode, r.stderr[-3000:])
    assert bad <= VALUES, bad


def test_bscan_tv_tiles_by_rounds(stub):
    """64 x 72 tiles, two to a CU, but where they just miss a round that the 64 x 128 ones keep."""
    out = run_child(stub, r"""
D = ctypes.c_double
for nz, nx, batch, inner, waves in [(2048, 1000, 1, 10, 8), (1024, 512, 8, 10, 8), (512, 64, 1, 10, 8), (2048, 1000, 1, 16, 16),
                                    (600, 1890, 1, 10, 16), (1280, 384, 1, 18, 16), (45, 540, 14, 10, 16), (36, 252, 14, 22, 16)]:
    p = plan(nz, nx, nz, batch=batch)
    st, names = kernels(lib.oct_prox, p, 1, D(0.1), D(1.0), inner, 1, D(0.0), BUF, P(8192), None, None)
    assert st == 0 and len(names) == 1 and f"Li{waves}E" in names[0], (nz, nx, inner, names)
    lib.oct_plan_destroy(p)
print("ok")
""")
    assert out.strip() == "ok"
