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
    """No launch leaves more than an eighth of the CUs idle, and none has more workgroups than there are CUs, each of which a workgroup takes whole."""
    run(tmp_path, """
    for (int per_strip = 1; per_strip <= 1024; ++per_strip)
        for (long long strips : {1LL, 255LL, 256LL, 820LL, 8192LL, 1LL << 20, 1LL << 26}) {
            const int used = wide_walkers(per_strip) * per_strip;
            if (used > WIDE_CUS || (wide_even(per_strip, strips) && used < 28)) { std::printf("%d: %d of %d", per_strip, used, WIDE_CUS); return 1; }
            if (used == WIDE_CUS && strips == 8192 && !wide_even(per_strip, strips)) { std::printf("%d fills them", per_strip); return 1; }
        }""")
