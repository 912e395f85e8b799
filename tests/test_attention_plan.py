"""Which sequences the decode attention takes together (no GPU): the limits of the form, the measured times that decide, and
that nothing but the call's sizes does."""
import ctypes
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2511_20100_amd", "csrc")


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, lib = str(d / "plan.cpp"), str(d / "plan.so")
    with open(src, "w") as f:
        f.write('#include "attention_plan.h"\nextern "C" int plan(int hd, int hq, int hkv, int B, int share, int p, int n) {\n'
                '  return mtmc::bf16::attention_sequences(hd, hq, hkv, B, share, p, n);\n}\n')
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I" + CSRC, src, "-o", lib], check=True)
    return ctypes.CDLL(lib).plan


HEADS = [(128, 16, 16), (128, 28, 4), (128, 16, 8), (64, 8, 8), (64, 32, 8), (128, 12, 2)]


@pytest.mark.parametrize("hd,hq,hkv", HEADS)
def test_limits_of_the_form(plan, hd, hq, hkv):
    for share in range(1, 33):
        for prompts in range(1, 128 // share + 1):
            for plen, new in ((1, 1), (16, 33), (512, 128), (701, 96), (4096, 4096)):
                B = prompts * share
                n = plan(hd, hq, hkv, B, share, plen, new)
                assert n >= 1 and share % n == 0 and n * (hq // hkv) <= 16 and n <= 8
                if B * hkv <= 256 or share == 1:
                    assert n == 1


def test_calls_of_the_bench_and_of_long_generations(plan):
    assert plan(128, 16, 16, 48, 4, 701, 96) == 4      # 31.0 us plain, 22.4 together
    assert plan(128, 28, 4, 128, 8, 1024, 48) == 2     # 27.3 and 20.9
    assert plan(128, 12, 2, 128, 8, 512, 1024) == 1    # 256 pairs: one round
    assert plan(64, 8, 8, 35, 7, 16, 512) == 1         # 5.0 plain, 11.0 together
    assert plan(128, 16, 8, 35, 7, 16, 512) == 1       # 12.6 and 22.5
    assert plan(128, 16, 16, 128, 8, 512, 33) > 1      # 54.4 and 20.4
