"""A property of the built code is kept once it is known, and only then: a query that failed
is made again (compiled here with g++, no GPU)."""
from __future__ import annotations

import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1409_4923_amd", "csrc")

SRC = r"""
#include "settled.hpp"
#include <cstdio>
enum Error { None = 0, Busy = 7 };
int main()
{
    for (int answer = 0; answer < 2; ++answer) {
        bm::Settled s;
        int asked = 0;
        auto ask = [&](bool &y) { ++asked; y = answer != 0; return asked < 3 ? Busy : None; };
        bool yes = answer == 0;
        for (int call = 1; call <= 5; ++call) {
            const Error e = s(yes, ask);
            if (e != (call < 3 ? Busy : None)) return 1;       // failed twice, then answered
            if (call >= 3 && yes != (answer != 0)) return 2;
        }
        if (asked != 3) return 3;                              // and not asked again
    }
    std::puts("ok");
    return 0;
}
"""


def test_only_answers_are_kept(tmp_path):
    src, exe = str(tmp_path / "t.cpp"), str(tmp_path / "t")
    with open(src, "w") as f:
        f.write(SRC)
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-Werror", "-I" + CSRC, src, "-o", exe])
    assert subprocess.run([exe], capture_output=True, text=True).stdout == "ok\n"


def test_launchers_use_it():
    """No launcher keeps the outcome of a HIP call by itself."""
    with open(os.path.join(CSRC, "launch.hpp")) as f:
        text = f.read()
    assert "static Settled" in text and "static const hipError_t" not in text
