"""Workspace layouts and the autotuner's cache on the host (tests/host_check/layouts.cpp, compiled here against the built library): no device."""
import os
import subprocess

import pytest

import paper_1809_10186_amd as qc

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    qc.lib()
    pkg = os.path.join(ROOT, "paper_1809_10186_amd")
    out = str(tmp_path_factory.mktemp("layouts") / "layouts")
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(pkg, "csrc"),
                    os.path.join(ROOT, "tests", "host_check", "layouts.cpp"), "-o", out,
                    os.path.join(pkg, "libqcoll.so"), "-L/opt/rocm/lib", "-lamdhip64",
                    "-Wl,-rpath," + pkg, "-Wl,-rpath,/opt/rocm/lib"], check=True)
    return out


@pytest.mark.parametrize("what", ["noalloc", "tune_key", "tune_schedule", "tune_fit"])
def test_layouts(driver, tmp_path, what):
    r = subprocess.run([driver, what, str(tmp_path / "cache.txt")], capture_output=True, text=True, timeout=300)
    print(r.stdout[-3000:], r.stderr[-1000:], flush=True)
    assert r.returncode == 0 and "layouts: ok" in r.stdout
