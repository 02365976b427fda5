"""Which passes of a step run on staged transforms, by grid, medium and the
caller's plans: the engine's selection on the CPU (tests/native/dispatch_test.cpp),
no kernel runs."""
import os
import shutil
import subprocess

import pytest

from paper_1408_4675_amd import _abi as A

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1408_4675_amd", "csrc")
NATIVE = os.path.join(ROOT, "tests", "native")
HIP_INCLUDE = "/opt/rocm/include"


@pytest.fixture(scope="module")
def route(tmp_path_factory):
    if shutil.which("g++") is None or not os.path.exists(os.path.join(HIP_INCLUDE, "hip")):
        pytest.skip("g++ or the HIP headers are missing")
    exe = str(tmp_path_factory.mktemp("dispatch") / "dispatch")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-D__HIP_PLATFORM_AMD__", "-I", HIP_INCLUDE,
                        "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                        os.path.join(NATIVE, "hip_host_stub.cpp"), os.path.join(NATIVE, "dispatch_test.cpp"),
                        "-o", exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout

    def run(shape, medium="maps", *args):
        r = subprocess.run([exe] + [str(n) for n in shape] + [medium] + list(args),
                           stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
        if r.stdout.startswith("error="):
            return dict(error=r.stdout)
        assert r.returncode == 0, r.stdout
        out = {}
        for word in r.stdout.split():
            k, v = word.split("=")
            out.setdefault("status", [])
            if k == "status":
                out["status"].append(int(v))
            else:
                out[k] = int(v)
        return out
    return run


STAGED = ("zs", "zs_skip", "ys", "xs", "xs_passes", "planes", "xs_adj")


# schedules of the 12- and 20-wide engines (and of the generic one) for lengths whose
# default is the generic engine; the last changes how even the x radices are
@pytest.mark.parametrize("shape,hint", [
    ((40, 100, 12), "hint:1:10,10:0"), ((40, 100, 12), "hint:1:20,5:8"), ((160, 160, 12), "hint:1:20,4,2:0"),
    ((200, 90, 20), "hint:0:10,10:0"), ((160, 160, 40), "hint:0:20,4:0"), ((160, 160, 40), "hint:2:20,2:0"),
    ((250, 135, 20), "hint:0:5,5,5:0")])
@pytest.mark.parametrize("medium", ["maps", "water", "lossless"])
def test_a_hint_leaves_staged_passes(route, shape, hint, medium):
    want, got = route(shape, medium), route(shape, medium, hint)
    assert want["ys"] or want["xs_passes"]
    assert got["status"] == [0]
    assert {k: got[k] for k in STAGED} == {k: want[k] for k in STAGED}


# an axis' own passes go to the engines, those of the others stay: x rows and a staged y
# pass (generic lengths), planes (two axes in one pass), powers of two
@pytest.mark.parametrize("shape", [(250, 135, 20), (100, 90, 12), (30, 8, 6), (64, 64, 48), (128, 36, 30)])
@pytest.mark.parametrize("medium", ["maps", "lossless"])
def test_a_forced_axis_leaves_the_others(route, shape, medium):
    want = route(shape, medium)
    for axis in range(3):
        got = route(shape, medium, "set:%d::0" % axis)
        assert got["status"] == [0]
        assert got["zs"] == (0 if axis == 2 else want["zs"])
        assert got["ys"] == (0 if axis == 1 else want["ys"])
        if axis == 2:
            assert {k: got[k] for k in STAGED[1:]} == {k: want[k] for k in STAGED[1:]}
            continue
        assert got["planes"] == 0
        rows = want["eng_x"] < 2 and axis == 1                 # generic x lengths have rows
        assert bool(got["xs_passes"]) == rows
    # a refused schedule changes nothing
    got = route(shape, medium, "set:1:7,11:0")
    assert got["status"] != [0] and {k: got[k] for k in STAGED} == {k: want[k] for k in STAGED}


YF, YI, ZG, ZD, ZA, XV, XD, XE = (1 << i for i in range(8))
X = XV | XD | XE


# what kw_routes says: the classes on engines, on staged transforms and on planes
@pytest.mark.parametrize("shape,medium,plans,engines,staged,planes", [
    ((30, 8, 6), "maps", [], 0, YF | ZG | ZD | ZA | X, 7),
    ((30, 8, 6), "lossless", [], 0, YF | ZG | ZD | XV | XD, 3),
    ((250, 135, 20), "maps", [], 0, 255, 0),
    ((250, 135, 48), "maps", [], 0, 255, 1),
    ((250, 135, 20), "lossless", [], 0, YF | YI | ZG | ZD | XV | XD, 0),
    ((64, 64, 256), "water", [], YF | ZG | ZA, ZD | X, 7),
    ((512, 64, 64), "water", [], YF | YI | XD | XE, ZG | ZD | ZA | XV, 1),
    ((30, 8, 6), "maps", ["set:0::0"], X, YF | YI | ZG | ZD | ZA, 0),
    # 32 points along z: 32 and 16 MiB of spectrum, and less
    ((512, 512, 32), "water", [], 255, 0, 0),
    ((512, 256, 32), "water", [], YF | YI | ZD | ZA | X, ZG, 0),
    ((512, 128, 32), "water", [], YF | YI | X, ZG | ZD | ZA, 0),
    ((250, 135, 20), "maps", ["set:2::0", "hint:1:9,15:0"], ZG | ZD | ZA, YF | YI | X, 0),
])
def test_routes_name_every_class_once(route, shape, medium, plans, engines, staged, planes):
    assert route(shape, medium, *plans)["routes"] == engines | staged << 8 | planes << 16


@pytest.mark.parametrize("axis,default_ms,is_forced", [(0, 12.0, True), (0, 9.0, False), (1, 9.1, False), (2, 12.0, True)])
def test_the_tuner_times_the_defaults_too(monkeypatch, tmp_path, axis, default_ms, is_forced):
    """A schedule is forced only where the step with it beats the step on the library's
    defaults; a step of the stand-in timings takes 9 ms with the best schedule."""
    from paper_1408_4675_amd import autotune as T
    from paper_1408_4675_amd import scenarios as sc
    scen = sc.small_case(24, 20, 18, seed=0)
    best = T.candidates(axis, T.lengths(scen.grid)[axis])[-1]

    def timed(scen, ax, sched, tile, steps):
        if ax is None:
            return dict.fromkeys(A.KERNEL_CLASSES, default_ms / 8)
        ms = dict.fromkeys(A.KERNEL_CLASSES, 9.0 / 8)
        if (sched, tile) != best:
            ms[T.AXIS_CLASSES[ax][0]] += 1.0
        return ms
    monkeypatch.setattr(T, "_time_plan", timed)
    monkeypatch.setenv(T.CACHE_ENV, str(tmp_path / "cache.json"))
    found = T.tune(scen, axes=(axis,), verbose=False)
    assert found[axis][:2] == best
    assert T.lookup(scen.grid) == {axis: best}
    assert T.forced(scen.grid) == ({axis} if is_forced else set())


@pytest.mark.parametrize("limit", [48 * 1024, 64 * 1024, 160 * 1024])
@pytest.mark.parametrize("nz", [18, 64, 81, 128, 160, 192, 225, 256, 375, 486, 512, 900])
def test_z_tiles_fit_the_lds_of_a_block(route, nz, limit):
    """Every launch of the staged z pass: the gradient's three tiles too."""
    for medium in ("maps", "water"):
        got = route((40 if nz < 300 else 8, 6, nz), medium, "lds=%d" % limit)
        if got["status"] != [0] or not got["zs"]:
            continue                                          # refused, or on the engines
        assert max(got["lds_grad"], got["lds_div"], got["lds_absm"]) <= limit
    if limit == 64 * 1024:
        assert got["zs"]


@pytest.mark.parametrize("name,cls", [
    ("kw_ystaged<true>(kw::(anonymous namespace)::YSArgs)", "ypass_inv"),
    ("kw_ystaged<false>(kw::(anonymous namespace)::YSArgs)", "ypass_fwd"),
    ("kw_zstaged<65812ull, 0, 3>(kw::(anonymous namespace)::ZSArgs)", "zfused_grad"),
    ("kw_zstaged<104316ull, 5, 1>(kw::(anonymous namespace)::ZSArgs)", "zfused_abs"),
    ("kw_xden_s<104316ull, 382ull, 6012ull, false, true>(kw::(anonymous namespace)::XSArgs)", "xden"),
])
def test_profiled_names_of_staged_kernels(name, cls):
    from paper_1408_4675_amd.profiling import kernel_class
    assert kernel_class("void kw::(anonymous namespace)::" + name) == cls


def test_lengths_of_the_staged_cases(route):
    """Which lengths of the GPU cases of the staged passes have stages: all columns but 625
    (5^4, no three radices up to 16), all packed rows but 243, 405 and 500 (the update's
    registers hold radices up to 8 in the first stages, 12 in the last)."""
    from tests.test_gpu_staged import COLUMNS, ROWS
    assert [n for n in COLUMNS if not route((8 if n > 64 else 40, 6, n))["zs"]] == [625]
    generic = [n for n in COLUMNS if route((8, n, 5))["eng_y"] < 2]
    assert [n for n in generic if not route((8, n, 5))["ys"]] == [625]
    assert [m for m in ROWS if not route((2 * m, 6 if m < 200 else 5, 5))["xs_passes"]] == [243, 405, 500]


def test_rows_without_stages(route):
    """The packed row lengths (nx = 2 m) whose x passes run on the engines for want of stages."""
    def smooth(n):
        for p in (2, 3, 5):
            while n % p == 0:
                n //= p
        return n == 1
    routes = {m: route((2 * m, 5, 5)) for m in range(200, 1025) if smooth(m)}
    assert [m for m, r in routes.items() if "error" in r] == [675, 729, 810]      # (the engines' density pass)
    none = [m for m, r in routes.items() if "error" not in r and not r["xs_passes"]]
    assert none == [243, 375, 405, 450, 486, 500, 540, 600, 625, 648, 720, 750, 800, 864, 900, 960, 972, 1000, 1024]
