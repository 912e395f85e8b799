"""Who may have a persistent launch under way, whether its workgroups are all there, and that they share out all of the work (no
GPU: the runtime's answers are made up by the first check, the second one's workgroups are threads)."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2511_20100_amd", "csrc")


def _run(tmp_path, name, *sources):
    exe = str(tmp_path / name)
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-Wall", "-Werror", "-Wno-unknown-pragmas", "-fsanitize=address,undefined", "-pthread",
                    "-D__HIP_PLATFORM_AMD__", "-isystem", "/opt/rocm/include", "-I" + CSRC, os.path.join(HERE, name + ".cpp"),
                    *sources, "-o", exe], check=True)
    run = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0 and run.stdout.strip() == "ok", run.stdout + run.stderr


def test_one_turn_and_none_while_launches_may_be_under_way(tmp_path):
    _run(tmp_path, "persistent_turn_check", "-x", "c++", os.path.join(CSRC, "persistent_turn.hip"))


def test_a_launch_runs_with_all_of_its_workgroups_or_with_those_on_the_list(tmp_path):
    _run(tmp_path, "roll_call_check")


def test_the_workgroups_of_a_step_share_out_all_of_its_work(tmp_path):
    _run(tmp_path, "persistent_cut_check")
