"""When the wave that streams a decode row's last 32-key block may rewrite the page of the row's new token by itself: only if every
slot of that page up to the token lies in that block.  The rule the kernels use, compiled for the host, against the definition."""
import os
import subprocess

from paper_2602_14516_amd.build import CSRC

SRC = r"""
#include <cstdio>
#include "plan.h"
int main() {
    for (int P = 16; P <= 64; P *= 2)
        for (int C = 0; C < 512; ++C)
            for (int begin = 0; begin <= C; begin += 64) {          // pieces of a row start at multiples of 64 keys
                const int last = (C - begin) / 32;
                bool alone = true;
                for (int t = C / P * P; t <= C; ++t) alone = alone && t >= begin && (t - begin) / 32 == last;
                if (ampd::page_in_last_block(C, P) != alone) {
                    std::printf("P %d C %d piece from %d: %d\n", P, C, begin, (int)alone);
                    return 1;
                }
            }
    return 0;
}
"""


def test_page_in_last_block_is_the_definition(tmp_path):
    src, exe = tmp_path / "rule.cpp", tmp_path / "rule"
    src.write_text(SRC)
    subprocess.check_call(["g++", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


def test_without_the_rule_a_large_page_is_shared(tmp_path):
    src, exe = tmp_path / "rule.cpp", tmp_path / "rule"
    src.write_text(SRC.replace("ampd::page_in_last_block(C, P)", "true"))
    subprocess.check_call(["g++", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 1 and r.stdout.startswith("P 64 C 32 "), r.stdout
