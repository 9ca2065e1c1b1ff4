"""The pool of pinned host buffers behind measure() and the spin copies: a
call takes the smallest buffer that fits, and small ones that fill the pool
give way to large ones (else every later read() pays for its own).  The rule
needs no GPU: a C++ program drives it."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_pool(tmp_path):
    exe = str(tmp_path / "pinned_pool")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-pthread",
                    "-I", os.path.join(ROOT, "paper_2502_18624_amd", "csrc"),
                    os.path.join(ROOT, "tests", "pinned_pool.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
