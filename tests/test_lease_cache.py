"""The bookkeeping of the cached decode-step graphs (no GPU): which entry makes room for another, and that none is
destroyed while a thread holds it or work that uses it is queued."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2511_20100_amd", "csrc")


def test_entries_outlive_their_use(tmp_path):
    exe = str(tmp_path / "lease_cache_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-Wall", "-Werror", "-fsanitize=address,undefined", "-pthread", "-I" + CSRC,
                    os.path.join(HERE, "lease_cache_check.cpp"), "-o", exe], check=True)
    run = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0 and run.stdout.strip() == "ok", run.stdout + run.stderr
