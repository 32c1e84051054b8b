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
