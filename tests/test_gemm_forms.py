"""The short GEMM forms and the rule that picks one, checked on the host (tests/gemm_forms_check.cpp)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_forms_and_choice(tmp_path):
    exe = os.path.join(str(tmp_path), "gemm_forms_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I",
                    os.path.join(ROOT, "paper_2504_12526_amd", "csrc"), "-o", exe,
                    os.path.join(ROOT, "tests", "gemm_forms_check.cpp")], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and ": ok" in r.stdout, r.stdout + r.stderr
