"""The multi-view adjoint's order of slots and passes (view_queue.hpp), built
for the host: no queued view's slot is overwritten, no pass takes more views
than its arrays hold, and the groups that the gradients are summed in are
those of a pass per group, for up to 40 views and two changes of the render
time at any of them."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_slots_and_groups(tmp_path):
    exe = str(tmp_path / "view_queue_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2311_18561_amd", "csrc"), "-o", exe,
                    os.path.join(ROOT, "tests", "host", "view_queue_check.cpp")], check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "view queue ok" in r.stdout
