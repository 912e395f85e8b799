"""Who may have a persistent launch under way (no GPU: the runtime's answers are made up by the check)."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2511_20100_amd", "csrc")


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("turn") / "persistent_turn_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-Wall", "-Werror", "-fsanitize=address,undefined", "-pthread",
                    "-D__HIP_PLATFORM_AMD__", "-isystem", "/opt/rocm/include", "-I" + CSRC,
                    os.path.join(HERE, "persistent_turn_check.cpp"), "-x", "c++", os.path.join(CSRC, "persistent_turn.hip"),
                    "-o", exe], check=True)
    return exe


def test_one_turn_and_none_while_launches_may_be_under_way(check):
    run = subprocess.run([check], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0 and run.stdout.strip() == "ok", run.stdout + run.stderr
