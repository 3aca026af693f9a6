"""Host-side decisions of the built library on the CPU: a child process loads it
with tests/hostcheck/hipstub.cpp in place of the HIP runtime ("device" memory is host
memory, no kernel runs) and tests/hostcheck/inject.cpp, which records launches and can
make an event wait fail."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.join(ROOT, "tests", "hostcheck")

PRELUDE = """
import ctypes as C
import sys
import numpy as np
stub = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)      # before the library: its HIP calls resolve here
from paper_1909_02894_amd import dirac as D
stub.inject_launch_fn.restype = C.c_void_p
stub.inject_launch_grid.restype = C.c_uint


def solver(n1, n2, prec=0, kind="curved", scheme=0, pml=None):
    pml = (0 if kind == "flat" else 2) if pml is None else pml
    g, m, p, _ = D.make_structs(n1, n2, 20.0, 20.0, 1e-4, 1.0, 0.5, metric=0 if kind != "curved" else 1,
                                spin=0 if kind != "curved" else 2, bump_A=1.0, bump_s=3.0, pml_width=pml)
    sc = D.Scheme(scheme, 0, 0, 0, 0.0)
    nb = D.footprint_bytes_ex(g, m, p, prec, sc, None)
    buf = np.zeros(nb, np.uint8)
    h = D.create_solver(g, m, p, prec, sc, None, buf.ctypes.data, nb, None)
    D.set_initial_spinor(h, np.zeros((n2, n1, 2), np.complex128))
    return h, buf


def store_mode(h):
    v = C.c_int32(-1)
    assert D.lib.dirac_get_store_mode(h, C.byref(v)) == 0
    return v.value


def schedule(h, d):
    s = D.Schedule()
    assert D.lib.dirac_get_schedule(h, d, C.byref(s)) == 0
    return s.radix, s.lines_per_wg, s.components_per_thread
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    if not (shutil.which("g++") and os.path.isdir("/opt/rocm/include/hip")):
        pytest.skip("no toolchain")
    lib = str(tmp_path_factory.mktemp("stub") / "libstub.so")
    cc = ["g++", "-shared", "-fPIC", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-w"]
    objs = []
    for f, extra in (("hipstub.cpp", ["-DhipLaunchKernel=stub_hipLaunchKernel",
                                      "-DhipEventSynchronize=stub_hipEventSynchronize"]), ("inject.cpp", [])):
        objs.append(lib + "." + f + ".o")
        subprocess.run([*cc, *extra, "-c", os.path.join(HERE, f), "-o", objs[-1]], check=True)
    subprocess.run([*cc, *objs, "-o", lib], check=True)

    def child(script):
        r = subprocess.run([sys.executable, "-c", PRELUDE + script, lib], cwd=ROOT, capture_output=True,
                           text=True, timeout=300)
        assert r.returncode == 0, (r.stdout[-2000:], r.stderr[-3000:])
    return child


def test_scheme1_has_no_store_mode(run):
    # the mask that dirac_set_store_mode refuses for Scheme I is not reported either
    run("""
h, buf = solver(64, 64, scheme=D.SCHEME_CN_GMRES)
assert store_mode(h) == 0, store_mode(h)
assert D.lib.dirac_set_store_mode(h, 1) == -1
""")


@pytest.mark.parametrize("waits", [0, 3, 9])
def test_failed_tuning_leaves_the_solver_as_it_was(run, waits):
    run(f"""
for kind, chosen in (("curved", None), ("flat", (1, (8, 1, 1), (8, 4, 1)))):
    h, buf = solver(256, 128, kind=kind)
    assert store_mode(h) == 3
    if chosen:
        assert D.lib.dirac_set_store_mode(h, chosen[0]) == 0
        for d in (0, 1):
            s = D.Schedule(*chosen[1 + d])
            assert D.lib.dirac_set_schedule(h, d, C.byref(s)) == 0
    before = store_mode(h), schedule(h, 0), schedule(h, 1)
    stub.inject_failing_wait({waits})
    assert D.lib.dirac_autotune(h, 2) == -5
    stub.inject_failing_wait(-1)
    assert (store_mode(h), schedule(h, 0), schedule(h, 1)) == before, (before, store_mode(h), schedule(h, 0))
    assert D.lib.dirac_autotune(h, 2) == 0
""")


def test_every_shape_has_a_default_schedule(run):
    # each length, direction, mode and precision from 16 lines on, through the line
    # counts where the defaults change; what is chosen is one of the compiled schedules
    run("""
for prec, top in ((0, 4096), (1, 8192)):
    for n in (16, 32, 64, 128, 256, 512, 1024, 2048, 4096, 8192):
        for other in (16, 64, 256):
            for d in (0, 1):
                n1, n2 = (n, other) if d == 0 else (other, n)
                for kind in ("flat", "layer", "curved"):
                    if n > top:
                        continue
                    h, buf = solver(n1, n2, prec, kind)
                    for dd, ln in ((0, n1), (1, n2)):
                        assert schedule(h, dd) in D.schedules(ln, prec, dd)
                    D.step_n(h, 1)
                    assert D.lib.dirac_destroy(h) == 0
""")


def test_which_column_launches_stream(run):
    # a streamed launch has 256 workgroups and a kernel of its own; below its least tile
    # count (256, flat 257) and for flat FP64 the same schedule launches a workgroup per tile
    run("""
def column_launch(n1, n2, prec, kind, sy):
    h, buf = solver(n1, n2, prec, kind)
    s = D.Schedule(*sy)
    assert D.lib.dirac_set_schedule(h, 1, C.byref(s)) == 0
    D.step_n(h, 1)                       # the x launch, then the y launch
    r = stub.inject_launch_fn(1), stub.inject_launch_grid(1)
    assert D.lib.dirac_destroy(h) == 0
    return r


cases = [(0, 2048, (16, 2, 2), 512, {"layer": True, "curved": True, "flat": False}),
         (0, 2048, (16, 2, 2), 1024, {"layer": True, "curved": True, "flat": False}),
         (1, 4096, (16, 2, 2), 512, {"layer": True, "curved": True, "flat": False}),
         (1, 4096, (16, 2, 2), 1024, {"layer": True, "curved": True, "flat": True}),
         (1, 2048, (16, 4, 2), 1024, {"layer": True, "curved": True, "flat": False}),
         (1, 2048, (16, 4, 2), 2048, {"layer": True, "curved": True, "flat": True}),
         (1, 4096, (16, 2, 1), 1024, {"layer": False, "curved": False, "flat": False}),
         (1, 2048, (16, 4, 1), 2048, {"layer": False, "curved": False, "flat": False})]
for prec, n2, sy, n1, modes in cases:
    for kind, streams in modes.items():
        plain = column_launch(n1 // 4, n2, prec, kind, sy)
        assert plain[1] == n1 // 4 // sy[1]
        fn, grid = column_launch(n1, n2, prec, kind, sy)
        assert (fn != plain[0]) == streams and grid == (256 if streams else n1 // sy[1]), (prec, n1, n2, kind, grid)
""")


def test_default_store_modes(run):
    # the defaults dirac.h states, by shape
    run("""
for n1, n2, prec, scheme, mode in ((64, 64, 0, 0, 3), (512, 512, 0, 0, 3), (1024, 1024, 0, 0, 1), (1024, 1024, 1, 0, 3),
                                   (2048, 1024, 0, 0, 0), (4096, 16, 0, 0, 0), (4096, 64, 1, 0, 0), (64, 512, 0, 0, 1),
                                   (256, 512, 0, 0, 3), (2048, 256, 1, 0, 3), (16, 2048, 1, 0, 1),
                                   (512, 1024, 1, D.SCHEME_EXP_SPLIT_2BIS, 1), (512, 512, 0, D.SCHEME_EXP_SPLIT_2BIS, 3)):
    h, buf = solver(n1, n2, prec, scheme=scheme)
    assert store_mode(h) == mode, (n1, n2, prec, scheme, store_mode(h))
    assert D.lib.dirac_destroy(h) == 0
""")


def test_defaults_of_8192_point_columns(run):
    # one line per workgroup until there are enough of them (grids of many lines take
    # gigabytes: their side of the rule is timed and tested on the GPU)
    run("""
for kind in ("flat", "layer", "curved"):
    for n1 in (16, 64, 256, 512):
        h, buf = solver(n1, 8192, 1, kind)
        assert schedule(h, 1) == ((16, 2, 2) if kind == "curved" and n1 >= 512 else (16, 1, 2)), (kind, n1)
        assert D.lib.dirac_destroy(h) == 0
""")


def test_store_modes_of_potentials_inside_the_direction_kernels(run):
    run("""
for n1, n2, prec, inside, apart in ((512, 1024, 0, 0, 3), (2048, 256, 0, 0, 3), (1024, 1024, 0, 0, 1), (512, 512, 0, 1, 3),
                                    (1024, 256, 0, 3, 3), (1024, 1024, 1, 1, 3), (2048, 256, 1, 3, 3)):
    V = np.zeros((n2, n1))
    g, m, p, _ = D.make_structs(n1, n2, 20.0, 20.0, 1e-4, 1.0, 0.5)
    em, keep = D.make_em(n1, n2, V=V)
    sc = D.Scheme(0, 0, 0, 0, 0.0)
    buf = np.zeros(D.footprint_bytes_ex(g, m, p, prec, sc, em), np.uint8)
    h = D.create_solver(g, m, p, prec, sc, em, buf.ctypes.data, buf.size, None)
    for form, mode in ((1, inside), (2, apart)):
        assert D.lib.dirac_set_potential_form(h, form) == 0
        assert store_mode(h) == mode, (n1, n2, prec, form, store_mode(h))
    assert D.lib.dirac_destroy(h) == 0
""")
