"""Which kernel a decode call goes to: the library's rule (csrc/anszp_choose.h) compiled for the host."""
import functools
import os
import shutil
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

DRIVER = r"""
#include <cstdio>
#include "anszp_choose.h"
int main() {
    unsigned table_log, streams, dtype, tables, mode, planned, cus, scales;
    unsigned long long chunks, words, elems;
    while (std::scanf("%u %u %u %u %llu %llu %llu %u %u %u %u", &table_log, &streams, &dtype, &tables, &chunks, &words, &elems, &scales, &mode, &planned, &cus) == 11) {
        anszp_decode_args_t a{};
        const float scale = 1.0f;
        a.table_log = table_log; a.n_streams = streams; a.out_dtype = dtype; a.n_tables = tables;
        a.n_chunks = chunks; a.payload_words = words; a.out_elems = elems;
        if (scales) { a.scales = &scale; a.n_scales = 1; }
        const LaunchChoice k = choose_kernel(a, int(mode), planned != 0, cus);
        // (in the order in which the kernels are looked for at a launch)
        if (k.waves.waves) std::puts("waves");
        else if (k.few) std::printf("few %u\n", k.few);
        else if (k.split) std::puts("split");
        else if (k.byte_table) std::puts("byte table");
        else if (k.stepwise) std::puts(k.streaming ? "streaming" : k.shared ? "stepwise shared" : "stepwise");
        else std::puts(k.small ? "look-ahead small" : "look-ahead large");
    }
    return 0;
}
"""


def compile_host(source, tmp, name):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    src, exe = os.path.join(tmp, name + ".cpp"), os.path.join(tmp, name)
    with open(src, "w") as f:
        f.write(source)
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-Wall", "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(ROOT, "paper_2406_06237_amd", "csrc"), src, "-o", exe])
    return exe


@functools.lru_cache(None)
def _exe():
    return compile_host(DRIVER, tempfile.mkdtemp(), "choice")


def kernel_of(host, planned=False, mode=0, cus=256):
    """The kernel that a HostContainer's decode goes to on a device of `cus` CUs."""
    dtype = {"u8": 0, "f32": 1, "bf16": 2}[host.out_dtype]
    call = (host.table_log, host.n_streams, dtype, len(host.layers), len(host.chunks), len(host.payload), host.numel, int(len(host.scales) > 0), mode, int(planned), cus)
    r = subprocess.run([_exe()], input=" ".join(map(str, call)), capture_output=True, text=True, timeout=60)
    assert r.returncode == 0
    return r.stdout.strip()
