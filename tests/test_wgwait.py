"""The workgroup's wait of the inserting kernel (csrc/lpht_wgwait.h), run on
threads: every wavefront gets what the first one's poll returned, and when some
wavefront has ended before a wait (its bound passed while it had nothing left to
do), the rest of the workgroup learns that the wait failed, also when it was the
polling one."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_waits_end_when_a_wavefront_has_left(tmp_path):
    exe = tmp_path / "wgwait"
    subprocess.run(["g++", "-std=c++20", "-O1", "-Wall", "-pthread", "-o", str(exe),
                    "-I", os.path.join(ROOT, "paper_1601_04017_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "wgwait.cpp")], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=60).stdout
    rows = {int(r[0]): [int(x) for x in r[1:]] for r in (line.split() for line in out.splitlines())}
    assert rows[-1] == [2, 4] * 4
    for leaver in range(4):
        # a first wait that all made, then a failed one (the leaver made none)
        assert rows[leaver] == [2, 0] * 4
