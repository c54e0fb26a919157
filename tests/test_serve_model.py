"""The serving loop's copies (csrc/lpht_server.cpp) over a model of HIP and of
the tables on the CPU (tests/native/serve_model.cpp): which arrays the copy
kernel takes, and that no operation runs when the arrays did not arrive."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1601_04017_amd", "csrc")
OK, ERR_DEVICE = 0, -5


@pytest.fixture(scope="module")
def seen(tmp_path_factory):
    exe = tmp_path_factory.mktemp("serve") / "serve_model"
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include",
                    "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-o", str(exe),
                    os.path.join(CSRC, "lpht_server.cpp"), os.path.join(ROOT, "tests", "native", "serve_model.cpp")],
                   check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=60).stdout
    return {k: int(v) for k, v in (line.split() for line in out.splitlines())}


@pytest.mark.parametrize("name,kernel_arrays,copies", [("pinned", 4, 0), ("device", 4, 0), ("other_device", 0, 4),
                                                       ("after_it", 4, 0), ("pageable", 0, 4)])
def test_arrays_arrive(seen, name, kernel_arrays, copies):
    assert seen[name + ".status"] == OK and seen[name + ".batches"] == 1
    assert (seen[name + ".kernel_arrays"], seen[name + ".copies"]) == (kernel_arrays, copies)


@pytest.mark.parametrize("name", ["copy_in_refused", "pageable_refused"])
def test_nothing_runs_on_arrays_that_did_not_arrive(seen, name):
    assert seen[name + ".status"] == ERR_DEVICE and seen[name + ".batches"] == 0
