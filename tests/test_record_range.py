"""The index ranges that the gradient gathers read (blend.hpp), built for the
host: no flag is read outside the flag array, whatever an overflowed sort left
in the index arrays."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_ranges_stay_inside_the_record_slots(tmp_path):
    exe = str(tmp_path / "record_range_check")
    subprocess.run(["/opt/rocm/bin/hipcc", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2311_18561_amd", "csrc"), "-o", exe,
                    os.path.join(ROOT, "tests", "host", "record_range_check.cpp")], check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "record range ok" in r.stdout
