"""Host check of the restriction's split of the test vectors over workgroups,
compiled and run on the CPU: no part is empty."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_no_part_of_the_restriction_is_empty(tmp_path):
    exe = tmp_path / "restrict_split_check"
    subprocess.run(["/opt/rocm/bin/hipcc", "-O1", "-std=c++17",
                    os.path.join(ROOT, "tests", "restrict_split_check.cpp"), "-o", str(exe)], check=True,
                   capture_output=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
    assert "SPLIT OK" in out.stdout
