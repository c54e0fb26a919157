"""The memory cache (csrc/lpht_pool.cpp) over a model of HIP on the CPU
(tests/native/pool_model.cpp): another thread's stream capture, a free that HIP
refuses, the bound on what is cached, and allocations that find no memory."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1601_04017_amd", "csrc")


@pytest.fixture(scope="module")
def seen(tmp_path_factory):
    exe = tmp_path_factory.mktemp("pool") / "pool_model"
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include",
                    "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-o", str(exe),
                    os.path.join(CSRC, "lpht_pool.cpp"), os.path.join(ROOT, "tests", "native", "pool_model.cpp")],
                   check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=60).stdout
    return {k: int(v) for k, v in (line.split() for line in out.splitlines())}


def test_capture_on_another_thread(seen):
    assert seen["capture_allocated"] and not seen["capture_harmed"]


def test_refused_free_keeps_the_block(seen):
    assert seen["kept_block_used_again"]


def test_bound_is_held_without_waiting(seen):
    assert seen["reserved_within_bound"] and seen["waits_over_bound"] == 0


def test_room_is_made_without_waiting_for_the_device(seen):
    assert seen["room_made"] and seen["waits_for_room"] == 0
    assert not seen["not_in_order"] and seen["in_order"] and not seen["never"]
    assert seen["waits_at_last"] == 0


def test_no_release_while_a_block_is_made(seen):
    assert seen["release_refused"]


def test_everything_is_released(seen):
    assert seen["released"] and seen["left"] == 0 and seen["events_left"] == 0
