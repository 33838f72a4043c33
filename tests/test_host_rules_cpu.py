"""Rules of the library's host side, and parts of its device code that the host can call, run on the
CPU from a host-only build of the library's sources (host_rules.hip)."""
from __future__ import annotations

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def host_rules(tmp_path_factory):
    if not os.path.exists(HIPCC) or shutil.which("g++") is None:
        pytest.skip("hipcc or g++ not available")
    tmp = tmp_path_factory.mktemp("host_rules")
    obj, stub, out = (str(tmp / f) for f in ("host_rules.o", "stub.cpp", "host_rules"))
    subprocess.check_call([HIPCC, "--offload-host-only", "-fuse-cuid=none", "-O1", "-std=c++17", "-fPIE",
                           "-Wno-unused-function", "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(ROOT, "paper_2507_03092_amd", "csrc"),
                           "-c", "-o", obj, os.path.join(ROOT, "tests", "host_rules.hip")])
    # (no kernel is launched: the place of the device code stays empty)
    with open(stub, "w") as f:
        f.write('extern "C" { extern const char __hip_fatbin[64]; const char __hip_fatbin[64] = {0}; }\n')
    lib = os.path.join(os.path.dirname(os.path.dirname(HIPCC)), "lib")
    subprocess.check_call(["g++", "-o", out, stub, obj, "-L", lib, "-lamdhip64", "-lpthread", f"-Wl,-rpath,{lib}"])
    return out


@pytest.mark.parametrize("check", ["list_by_step", "windows_of_a_layer", "list_ahead", "captures", "batch_waves", "noalloc_limit"])
def test_host_rule(host_rules, check):
    r = subprocess.run([host_rules, check], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-3000:] + r.stderr[-3000:]
