"""The arithmetic of the fused convolution's panel decoder (csrc/anszp_panel.h), checked exhaustively on the host by a
small native program built from the header itself."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2406_06237_amd", "csrc")


def _run(tmp_path, body):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "check.cpp", tmp_path / "check"
    src.write_text('#include <cstdio>\n#include "anszp_panel.h"\nint main() {\n' + body + '\n    std::puts("ok");\n    return 0;\n}\n')
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-Wall", "-I", CSRC, str(src), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout


def test_staged_words_are_read_inside_lds_whatever_the_stream_says(tmp_path):
    # `left` of a corrupt stream may be any number: the word and the one behind it stay in the LDS every launch has;
    # of a valid stream it stands for the word it counts, anywhere in the staging room
    _run(tmp_path, """
    for (uint32_t left = 0;; left += 8u) {
        const uint32_t a = stage_address(left);
        if ((a & 3u) != 0u || a + 8u > kLeastLds) { std::printf("left %u: address %u", left, a); return 1; }
        if (left < 8u * kStageBytes && a != left / 32u * 4u) { std::printf("left %u: address %u", left, a); return 1; }
        if (left == 0xFFFFFFF8u) break;
    }""")


def test_rows_of_a_chunks_elements_for_every_reduction_length(tmp_path):
    # pos / K for every K a panel may have and every element a look-up can reach in a chunk of up to 16 rows, with the
    # factors the 24-bit multiplication takes
    _run(tmp_path, """
    for (uint32_t K = 1; K <= 4608u; ++K) {
        const RowReciprocal r = row_reciprocal(K);
        const uint32_t reach = 16u * K + 8u * 64u;
        if (r.magic >= 1u << 24 || (uint64_t(reach) << r.shift) >= 1u << 24) { std::printf("K %u: factors", K); return 1; }
        uint32_t row = 0, next = K;
        for (uint32_t pos = 0; pos < reach; ++pos) {
            if (pos == next) { ++row; next += K; }
            if (uint32_t((uint64_t(pos << r.shift) * r.magic) >> 32) != row) { std::printf("K %u, element %u", K, pos); return 1; }
        }
    }""")
