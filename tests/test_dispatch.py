"""Which passes of a step run on staged transforms, by grid, medium and the
caller's plans: the engine's selection on the CPU (tests/native/dispatch_test.cpp),
no kernel runs."""
import os
import shutil
import subprocess

import pytest

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
