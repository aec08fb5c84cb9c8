"""The lazy Shoup product of the 64-bit integer butterflies against 128-bit integers (host build of the same header)."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_lazy_product_is_below_four_moduli_and_congruent(tmp_path):
    exe = str(tmp_path / "shoup_check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-o", exe, os.path.join(HERE, "shoup_check.cpp")], check=True)
    res = subprocess.run([exe], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout
