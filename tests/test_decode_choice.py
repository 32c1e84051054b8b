"""Which kernel decodes a call (csrc/anszp_choose.h), on the host over calls of every size: what one kernel takes over from another it
can hold."""
import subprocess

import pytest

import test_gpu_few as few
import test_gpu_plan as plan
from decode_choice import compile_host, kernel_of
from helpers import host_from_oracle, oracle_encode

DRIVER = r"""
#include <cmath>
#include <cstdio>
#include <random>
#include "anszp_choose.h"
#define REQUIRE(what) do { if (!(what)) { std::printf("%s: 2^%u states, %u streams, type %u, %llu chunks of %u layers, %llu words, %llu elements, planned %d, %u CUs: few %u", \
    #what, a.table_log, a.n_streams, a.out_dtype, (unsigned long long)a.n_chunks, a.n_tables, (unsigned long long)a.payload_words, (unsigned long long)a.out_elems, planned, cus, k.few); return 1; } } while (0)
int main() {
    std::mt19937 rng(1);
    auto upto = [&](double most) { return uint64_t(std::exp(std::uniform_real_distribution<double>(0.0, std::log(most + 0.999))(rng))); };
    uint32_t taken[5] = {};
    for (uint32_t i = 0; i < 400000u; ++i) {
        anszp_decode_args_t a{};
        a.table_log = 1u + rng() % 12u;
        a.n_streams = rng() % 2u ? 64u : 1u + rng() % 64u;
        a.out_dtype = rng() % 3u;
        a.n_chunks = upto(3000);
        a.n_tables = uint32_t(upto(double(a.n_chunks)));
        a.out_elems = a.n_chunks * upto(70000);
        a.payload_words = uint64_t(double(a.out_elems) * a.table_log / 32.0 * (rng() % 1000u) / 1000.0);
        const bool planned = rng() % 2u;
        const uint32_t cus = rng() % 4u ? 256u : 1u + rng() % 304u;
        const LaunchChoice k = choose_kernel(a, 0, planned, cus);
        if (!k.few || k.waves.waves) continue;
        ++taken[k.few <= 4u ? k.few : 0u];
        REQUIRE(!k.split && !k.stepwise && k.few <= kFewMostPerCu && k.few <= (a.n_chunks + cus - 1u) / cus);
        // so many workgroups are resident on a CU: LDS is given out in pieces of 1,280 bytes
        REQUIRE(k.few * ((few_lds(k.few) + 1279u) / 1280u * 1280u) <= 160u * 1024u && few_lds(k.few) % 16u == 0u);
        // the mean is all the rule sees of the chunks: any that the look-ahead kernel would hold has to fit
        REQUIRE(few_words(few_lds(k.few), a.table_log) >= int32_t(k.small ? SmallLds::kSoloWords : LargeLds::kSoloWords));
    }
    if (!taken[0] && taken[1] > 1000u && taken[2] > 1000u && taken[3] > 100u && taken[4] > 100u) std::puts("ok");
    return 0;
}
"""


def test_a_chunk_that_another_kernel_would_hold_fits(tmp_path):
    r = subprocess.run([compile_host(DRIVER, str(tmp_path), "sizes")], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout


@pytest.mark.parametrize("table_log,n_short,long,kernel", few.MANY_WORDS)
def test_the_gpu_tests_of_many_words_run_what_they_name(orc, table_log, n_short, long, kernel):
    w = few.many_words(table_log, n_short, long)
    h = host_from_oracle(oracle_encode(orc, w), w)
    words = int(h.chunks["payload_words"].max())
    assert kernel_of(h) == kernel and (9000 < words <= 11672 if table_log == 12 else 5500 < words <= 5912)


def _kernel(orc, w, planned=False):
    return kernel_of(host_from_oracle(oracle_encode(orc, w), w), planned)


@pytest.mark.parametrize("n_chunks,table_log,kernel", few.NUMBERS)
def test_numbers_of_chunks(orc, n_chunks, table_log, kernel):
    assert _kernel(orc, few.numbers_of_chunks(n_chunks, table_log)) == kernel


@pytest.mark.parametrize("n_layers,chunks,table_log,dtype,kernel", few.LAYERS)
def test_layers_of_few_chunks(orc, n_layers, chunks, table_log, dtype, kernel):
    assert _kernel(orc, few.layers_of_few_chunks(n_layers, chunks, table_log, dtype)) == kernel


def test_planned_calls(orc):
    workloads = plan._workloads()
    assert {name: _kernel(orc, workloads[name], True) for name in plan.KERNELS} == plan.KERNELS
