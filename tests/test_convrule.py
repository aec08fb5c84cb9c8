"""The rule that picks a basis conversion's kernel, over every size that a context can have (host build of the same header)."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_every_conversion_has_a_kernel_and_other_sizes_are_refused(tmp_path):
    exe = str(tmp_path / "convrule_check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-o", exe, os.path.join(HERE, "convrule_check.cpp")], check=True)
    res = subprocess.run([exe], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout
