"""Host-only check of which caller arrays kernels use in place: memory of the
device that the call runs on, never another device's (a kernel may fault there)
nor managed memory.  No path of the library asks the looser question (a pointer
a copy would take as device memory) before it hands a pointer to a kernel."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
INC = os.path.join(ROOT, "paper_2412_17132_amd", "csrc")


def test_rule_on_every_kind_of_pointer(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "pointers")
    build = subprocess.run([gxx, "-std=c++17", "-Wall", "-I", INC, os.path.join(ROOT, "tests", "pointers_driver.cpp"),
                            "-o", exe], capture_output=True, text=True)
    assert build.returncode == 0, build.stderr
    run = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0 and "all checks passed" in run.stdout, run.stdout


def test_in_place_users_ask_the_rule():
    """`is_device_ptr` decides the kind of a copy only, in `to_host`."""
    text = open(os.path.join(INC, "gwc_api.hip")).read()
    uses = [m.start() for m in re.finditer(r"\bis_device_ptr\(", text)]
    body = text[text.index("std::vector<T> to_host("):]
    body = body[:body.index("\n}\n")]
    assert len(uses) == 2 and body.count("is_device_ptr(") == 1  # its definition and to_host
