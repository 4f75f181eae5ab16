"""What the C ABI keeps between calls, when one of its HIP calls fails: capi.cpp
built for the host over a stand-in for the runtime and the launchers
(capi_host.cpp), one scenario a test (CPU)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_0904_0642_amd", "csrc")


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    d = tmp_path_factory.mktemp("capi")
    objs = []
    for src in (os.path.join(CSRC, "capi.cpp"), os.path.join(ROOT, "tests", "capi_host.cpp")):
        objs.append(str(d / (os.path.basename(src) + ".o")))
        r = subprocess.run(["hipcc", "-x", "hip", "--cuda-host-only", "-O1", "-std=c++17", "-w", "-I" + CSRC,
                            "-I" + os.path.join(ROOT, "include"), "-c", src, "-o", objs[-1]],
                           capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
    out = str(d / "capi_host")
    # no HIP library: the stand-in is all there is (the device code's symbol stays open)
    r = subprocess.run(["g++", "-no-pie", "-pthread", "-o", out] + objs + ["-Wl,--unresolved-symbols=ignore-all"],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return out


@pytest.mark.parametrize("scenario", ["failed_measurement", "failed_sweeps", "given_up_waits", "failed_clearing",
                                      "copies_behind_sweeps"])
def test_scenario(exe, scenario):
    r = subprocess.run([exe, scenario], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[:4000] + r.stderr
