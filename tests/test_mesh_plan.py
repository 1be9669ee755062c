"""The host plan of the near / far split (plain C++), over sizes and domains."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_plan(tmp_path):
    exe = str(tmp_path / "mesh_check")
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-o", exe,
                           os.path.join(ROOT, "tests", "mesh_check.cpp")])
    out = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stdout
