"""What the library's host code decides, asked on the CPU: tests/host_plan/driver.cpp compiled for the host alone."""
import functools
import os
import shutil
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@functools.lru_cache(maxsize=None)
def _driver():
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not found")
    out = tempfile.mkdtemp()
    exe = os.path.join(out, "host_plan_driver")
    # no device pass: the code object that the launch stubs refer to is missing, and nothing is launched
    cmd = [hipcc, "--offload-arch=gfx950", "--offload-host-only", "-O1", "-std=c++17", "-x", "hip",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"),
           os.path.join(ROOT, "tests", "host_plan", "driver.cpp"), "-o", exe, "-Wl,--unresolved-symbols=ignore-all"]
    build = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=600)
    assert build.returncode == 0, build.stdout[-4000:]
    with open(exe, "rb") as f:
        code = f.read()
    shutil.rmtree(out, ignore_errors=True)
    return code


def ask(queries):
    """One dict of integers per query."""
    out = tempfile.mkdtemp()
    try:
        exe = os.path.join(out, "host_plan_driver")
        with open(exe, "wb") as f:
            f.write(_driver())
        os.chmod(exe, 0o755)
        run = subprocess.run([exe], input="\n".join(queries) + "\n", stdout=subprocess.PIPE, stderr=subprocess.STDOUT,
                             text=True, timeout=120)
    finally:
        shutil.rmtree(out, ignore_errors=True)
    assert run.returncode == 0, run.stdout[-2000:]
    answers = [{k: int(v) for k, v in (p.split("=") for p in line.split())} for line in run.stdout.splitlines()]
    assert len(answers) == len(queries)
    return answers
