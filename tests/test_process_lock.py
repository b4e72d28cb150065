"""The lock by which one process at a time runs the one-kernel decoder on a GPU: held once, given back, not kept by a forked
child, refused where the system will not say."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_process_lock(tmp_path):
    exe = str(tmp_path / "check")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-pthread", os.path.join(ROOT, "tests", "process_lock_check.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe, f"specdec-check-{os.getpid()}"], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
