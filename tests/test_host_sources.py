"""The library's host sources on the CPU: program.cpp, dl_api.cpp and serve.cpp
compiled for the host alone and linked with a stand-in for the HIP runtime and
the kernel launches (tests/host/), for what needs no device: sizes and strides
that calls pass on, and what happens when memory runs out."""
from __future__ import annotations

import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1608_00139_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    out = tmp_path_factory.mktemp("host")
    sources = [os.path.join(CSRC, f) for f in ("program.cpp", "dl_api.cpp", "serve.cpp")]
    sources += [os.path.join(HERE, "host", f) for f in ("runtime.cpp", "driver.cpp")]
    jobs, objs = [], []
    for s in sources:
        objs.append(str(out / (os.path.basename(s) + ".o")))
        jobs.append(subprocess.Popen([HIPCC, "--offload-arch=gfx950", "--offload-host-only", "-x", "hip", "-O1", "-g",
                                      "-std=c++17", "-c", s, "-o", objs[-1]],
                                     stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True))
    for j in jobs:
        text, _ = j.communicate(timeout=240)
        assert j.returncode == 0, text
    exe = str(out / "driver")
    # launches that no case reaches stay undefined
    r = subprocess.run(["g++", *objs, "-o", exe, "-Wl,--unresolved-symbols=ignore-all", "-no-pie", "-lpthread"],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    return exe


@pytest.mark.parametrize("case", ["fetch_after_rebind", "kept_matrices_given_up", "host_memory_runs_out",
                                  "launch_tags"])
def test_case(driver, case):
    r = subprocess.run([driver, case], capture_output=True, text=True, timeout=60)
    assert (r.returncode, r.stdout) == (0, "ok\n"), (case, r.returncode, r.stdout, r.stderr)
