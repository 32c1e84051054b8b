"""How the fused convolution's sliced kernel is launched (csrc/anszp_conv_plan.h), checked on the host over calls of every
size: what the kernel takes for granted about tiles, slices and LDS, and that no few workgroups wait for a CU."""
import os
import shutil
import subprocess

import pytest

from decode_choice import compile_host

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

DRIVER = r"""
#include <cstdio>
#include <random>
#include "anszp_conv_plan.h"
#define REQUIRE(what) do { if (!(what)) { std::printf("%s: mode %u, %u x %u x %u x %u, rows %u, 2^%u states, %u tiles, %u CUs: %u row tiles, %u tiles, %u slices, %u of %u tiles, %u LDS", \
    #what, mode, a.cout, a.cin, a.kh, a.kw, a.rows_per_chunk, a.table_log, n_tiles, cus, p.mr, p.qt, p.k_groups, p.splits, p.tiles_per_split, p.lds_bytes); return 1; } } while (0)
int main() {
    std::mt19937 rng(1);
    auto upto = [&](double most) { return uint32_t(std::exp(std::uniform_real_distribution<double>(0.0, std::log(most + 0.999))(rng))); };
    for (uint32_t i = 0; i < 400000u; ++i) {
        anszp_conv_args_t a{};
        const uint32_t mode = 1u + rng() % 3u;
        a.kw = mode == kPoint ? 1u : 3u;
        a.kh = mode == kPoint ? 1u : 1u + rng() % 5u;
        a.cin = 32u * upto(kMaxK / (32u * a.kh * a.kw));
        if (rng() % 8u == 0u) a.cin = kMaxK / (a.kh * a.kw) / 32u * 32u;
        a.cout = 16u * upto(300);
        a.rows_per_chunk = 1u << rng() % 5u;
        a.table_log = 1u + rng() % 12u;
        a.x_layout = rng() % 2u; a.y_layout = rng() % 2u;
        a.y_dtype = rng() % 2u ? ANSZP_OUT_BF16 : ANSZP_OUT_F32;
        const uint32_t n_tiles = upto(1u << 27), cus = rng() % 4u ? 256u : 1u + rng() % 304u;
        const uint32_t K = a.cin * a.kh * a.kw, row_stride = ((K + 31u) & ~31u) + kRowPad, units = (mode == kPoint ? 1u : a.kh) * (a.cin / 32u);
        const SlicedPlan p = plan_sliced(a, mode, K, row_stride, n_tiles, cus);
        REQUIRE(p.mr == 1u || p.mr == 2u || p.mr == 4u);
        REQUIRE(a.cout % (kRows * p.mr) == 0u);
        const uint32_t n_mtiles = a.cout / (kRows * p.mr), elems = kRows * p.mr * row_stride, front = kStageBytes + (16u << a.table_log);
        // the decoded panel, widened if it is one of bytes, and the slices' sums fit what is asked for, and that the CU
        REQUIRE(p.lds_bytes <= kLdsLimit && front + elems * (p.p16 ? 2u : 1u) + 64u <= p.lds_bytes);
        REQUIRE(p.p16 || (2u * (elems + 64u) <= p.lds_bytes && elems + 64u <= kWidenPieces * kThreads * 16u));
        REQUIRE(p.k_groups >= 1u && kWaves % p.k_groups == 0u);
        const uint32_t t_groups = kWaves / p.k_groups;
        REQUIRE(p.qt >= 1u && p.qt <= most_tiles(p.mr, mode));
        REQUIRE(p.k_groups == 1u || (p.round_tiles == p.tiles_per_split && kWaves * p.qt * p.mr * 1024u <= p.lds_bytes && units >= p.k_groups));
        // every range of tiles has p.qt of them or one fewer, all rounds and splits together all of them
        REQUIRE(p.round_tiles >= 1u && (p.round_tiles + t_groups - 1u) / t_groups == p.qt);
        REQUIRE(p.slice_units * p.k_groups >= units);
        REQUIRE(uint64_t(p.splits) * p.tiles_per_split >= n_tiles && uint64_t(p.splits - 1u) * p.tiles_per_split < n_tiles);
        REQUIRE(uint64_t(n_mtiles) * p.splits < (1u << 22));
        // one workgroup per CU: with several shares a panel, one more each would make some wait for all others
        REQUIRE(n_mtiles > cus / 8u || n_mtiles * p.splits <= cus);
    }
    std::puts("ok");
    return 0;
}
"""


def _run(tmp_path, driver):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "plan.cpp", tmp_path / "plan"
    src.write_text("#include <cmath>\n" + driver)
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-Wall", "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(ROOT, "paper_2406_06237_amd", "csrc"), str(src), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout


def test_plans_of_every_size(tmp_path):
    _run(tmp_path, DRIVER)


def test_plans_of_channels_that_are_multiples_of_eight(tmp_path):
    """The last unit of a kernel row has fewer than 32 channels then: units are counted up, rows keep their padding."""
    driver = DRIVER.replace("a.cin = 32u * upto(kMaxK / (32u * a.kh * a.kw));", "a.cin = 8u * upto(kMaxK / (8u * a.kh * a.kw));")
    driver = driver.replace("a.cin = kMaxK / (a.kh * a.kw) / 32u * 32u;", "a.cin = kMaxK / (a.kh * a.kw) / 8u * 8u;")
    driver = driver.replace("a.kh) * (a.cin / 32u);", "a.kh) * ((a.cin + 31u) / 32u);")
    assert driver.count("8u * upto") == 1 and driver.count("/ 8u * 8u") == 1 and driver.count("+ 31u) / 32u)") >= 1
    _run(tmp_path, driver)


def test_plans_of_half_a_row_tile(tmp_path):
    """What holds for whole row tiles holds for panels of eight channels, which are of bf16 values always."""
    driver = DRIVER.replace("plan_sliced(a, mode,", "plan_half_tile(a, mode,").replace("p.mr == 1u || p.mr == 2u || p.mr == 4u", "p.rows == (p.rows == 8u ? 8u : 16u * p.mr)")
    driver = driver.replace("a.cout % (kRows * p.mr) == 0u", "a.cout % p.rows == 0u && p.rows % a.rows_per_chunk == 0u && (p.rows > 8u || (p.p16 && ++halves))")
    driver = driver.replace("a.cout / (kRows * p.mr), elems = kRows * p.mr * row_stride", "a.cout / p.rows, elems = p.rows * row_stride")
    driver = driver.replace("std::mt19937 rng(1);", "std::mt19937 rng(1); uint32_t halves = 0;").replace("std::puts", "if (halves > 2000u) std::puts")
    assert driver.count("halves") == 3 and driver.count("p.rows") >= 6
    _run(tmp_path, driver)


CALLS = r"""
#include <cmath>
#include <cstdio>
#include "anszp_conv_plan.h"
int main() {
    anszp_conv_args_t a{};
    while (std::scanf("%u %u %u %u %u %u %u %u %u %u %u", &a.cout, &a.cin, &a.kh, &a.kw, &a.batch, &a.in_h, &a.in_w, &a.stride, &a.pad, &a.rows_per_chunk, &a.x_layout) == 11) {
        a.y_layout = a.x_layout; a.y_dtype = ANSZP_OUT_F32; a.table_log = 12u;
        const uint32_t K = a.cin * a.kh * a.kw, out_h = (a.in_h + 2u * a.pad - a.kh) / a.stride + 1u, out_w = (a.in_w + 2u * a.pad - a.kw) / a.stride + 1u;
        std::printf("%u\n", plan_call(a, K, ((K + 31u) & ~31u) + kRowPad, out_h, out_w, a.batch, 256u).plan.rows);
    }
    return 0;
}
"""


def test_the_gpu_tests_of_half_a_row_tile_run_panels_of_eight_rows(tmp_path):
    import test_gpu_conv
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    exe = compile_host(CALLS, str(tmp_path), "calls")
    calls = [(*shape, *rest, layout) for shape, *rest in test_gpu_conv.HALF_TILES for layout in (0, 1)]
    r = subprocess.run([exe], input="\n".join(" ".join(map(str, c)) for c in calls), capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.split() == ["8"] * len(calls)
    assert {c[9] for c in calls} == {1, 2, 4, 8}
