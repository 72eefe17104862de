"""The sizes of pair_wide_kernel, gone through on the host: a program of plain C++ includes the header that the kernel and its launch take them from."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2408_11500_amd", "csrc")


def run(tmp_path, body):
    source, program = tmp_path / "t.cpp", tmp_path / "t"
    source.write_text('#include "wide_rules.h"\n#include <cstdio>\n#include <initializer_list>\nusing namespace slicegcn;\nint main() {\n' + body + "\nreturn 0; }\n")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(source), "-o", str(program)], check=True, timeout=120)
    r = subprocess.run([str(program)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout


def test_weights_requested_lie_in_lds(tmp_path):
    """The groups of four k that a strip's steps ask for ahead of time lie in the array."""
    run(tmp_path, """
    for (int nt = 2; nt <= 4; ++nt)
        for (int K = 4; K <= wide_k(nt); ++K)
            for (int c = 0; c * WIDE_CHUNK < K; ++c)
                for (int q = 0; q < WIDE_CHUNK / 8 && 8 * q < K - c * WIDE_CHUNK; ++q) {
                    const int last = c * (WIDE_CHUNK / 4) + 2 * (q + 1) + 1; // by the upper half of the lanes
                    if (wide_more(K - c * WIDE_CHUNK, q) && (last >= wide_groups(K) || last >= wide_groups(wide_k(nt)))) {
                        std::printf("nt %d K %d c %d q %d: %d of %d", nt, K, c, q, last, wide_groups(K));
                        return 1;
                    }
                }""")


def test_grids_fill_the_chip_once(tmp_path):
    """No launch leaves more than five of the 32 CUs that share an L2 idle, and none has more workgroups than there are CUs, each of which a workgroup takes whole."""
    run(tmp_path, """
    for (int per_strip = 1; per_strip <= 1024; ++per_strip)
        for (long long strips : {1LL, 255LL, 256LL, 820LL, 8192LL, 1LL << 20, 1LL << 26}) {
            const int used = wide_walkers(per_strip) * per_strip;
            const bool even = wide_even(per_strip, strips);
            if (used > WIDE_CUS || (even && used < 27)) { std::printf("%d: %d of %d", per_strip, used, WIDE_CUS); return 1; }
            if (used == WIDE_CUS && strips == 8192 && !even) { std::printf("%d fills them", per_strip); return 1; }
        }""")


def test_products_too_short_for_their_columns(tmp_path):
    """Kinds of shapes that are slower than by the general kernel on average, and beside them kinds that are faster: tiles a workgroup takes, workgroups along the
    columns, steps of k, rows that begin on whole lines, activation bits, two products."""
    slower = [(2, 5, 16, 1, 1, 0), (2, 7, 23, 1, 0, 1), (3, 1, 7, 0, 1, 0), (3, 5, 15, 0, 0, 0), (3, 6, 15, 1, 1, 0), (4, 2, 15, 0, 0, 0), (4, 8, 8, 0, 1, 0), (4, 5, 15, 1, 0, 0),
              (4, 2, 7, 1, 0, 0)]
    faster = [(2, 5, 24, 0, 0, 0), (2, 5, 128, 1, 0, 1), (2, 1, 96, 0, 1, 0), (3, 1, 16, 0, 0, 0), (3, 6, 48, 1, 0, 0), (3, 2, 130, 0, 0, 1), (4, 1, 8, 1, 0, 0), (4, 4, 4, 1, 1, 0),
              (4, 8, 16, 0, 0, 0), (4, 2, 160, 0, 1, 0), (3, 2, 4, 0, 1, 1)]
    table = lambda shapes: ", ".join("{%d, %d, %d, %d, %d, %d}" % s for s in shapes)
    run(tmp_path, """
    const int slower[][6] = {%s}, faster[][6] = {%s};
    for (auto &s : slower) if (wide_long(s[0], s[1], s[2], s[3], s[4], s[5])) { std::printf("%%d %%d %%d", s[0], s[1], s[2]); return 1; }
    for (auto &s : faster) if (!wide_long(s[0], s[1], s[2], s[3], s[4], s[5])) { std::printf("%%d %%d %%d", s[0], s[1], s[2]); return 1; }""" % (table(slower), table(faster)))
