"""The push ensemble kernel's numbering of words, on the host: for every shape
the planner lets through, every word's window and group against the division
they stand for."""
import subprocess

import paper_0908_3934_amd.build as build

PROGRAM = r"""
#include <cstdio>
#include <initializer_list>
#include "push_plan.h"
using namespace geonet;
int main() {
    long shapes = 0, wrong = 0;
    unsigned most = 0;
    for (int groups = 1; groups <= kWordMaxGroups; ++groups)
        for (int vertices : {groups * 64 - 63, groups * 64})
            for (int delay = 1; delay <= 255; ++delay) {
                const PushShape s = push_shape(vertices, delay, 152 * 1024);
                if (s.window < 1) continue;
                ++shapes;
                // the largest delay's window exists, and a delay within its window fits its bits
                if (s.n_win > kWordMaxWindows || (delay - 1) / s.window != s.n_win - 1 || s.window > 1 << (16 - s.tbits) ||
                    vertices > 1 << s.tbits || s.lds > 152 * 1024) ++wrong;
                const uint32_t inv = word_inverse(groups), words = uint32_t(s.n_win) * groups;
                most = words > most ? words : most;
                for (uint32_t k = 0; k < words; ++k) wrong += word_window(k, inv) != k / groups;
            }
    std::printf("%ld %ld %u\n", shapes, wrong, most);
}
"""


def test_words_of_every_shape(tmp_path):
    src, exe = tmp_path / "words.cpp", tmp_path / "words"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-I" + build.CSRC, str(src), "-o", str(exe)])
    shapes, wrong, most = map(int, subprocess.check_output([str(exe)]).split())
    assert shapes > 20000 and most > 8609 and wrong == 0
