"""Arenas and the server's slab cache, compiled for the host against a stand-in
for the HIP allocation calls (tests/host): what they keep, give back and report."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2507_06471_amd", "csrc")


def test_arena_bookkeeping(tmp_path):
    exe = str(tmp_path / "arena")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-Wall", "-Werror", "-fsanitize=address,undefined", "-I",
                    os.path.join(HERE, "host"), "-I", CSRC, os.path.join(HERE, "host", "arena.cpp"), "-o", exe],
                   check=True)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out.stdout + out.stderr
