"""GPU parity of decode_few (a workgroup per chunk, csrc/anszp_few.h) against the oracle, bit for bit: the calls anszp_decode
sends there by itself, at the sizes where it can go wrong."""
import numpy as np
import pytest
import torch

from paper_2406_06237_amd import binding as B
from paper_2406_06237_amd import workloads as W

from helpers import host_from_oracle, oracle_encode, oracle_expected

pytestmark = pytest.mark.gpu


def _check(orc, w, planned=False, out_dtype=None):
    c = oracle_encode(orc, w)
    if out_dtype:
        w.out_dtype = out_dtype
    _, expect = oracle_expected(orc, c, w)
    d = B.to_device(host_from_oracle(c, w))
    guard = 4096
    dt = getattr(torch, {"u8": "uint8", "f32": "float32", "bf16": "bfloat16"}[w.out_dtype])
    buf = torch.full((w.numel + 2 * guard,), 77, dtype=dt, device="cuda:0")
    out = buf[guard:guard + w.numel]
    args = B.decode_args(d, out)
    if planned:
        B.decode_planned_raw(args, B.plan_decode(args))
    else:
        B.decode_raw(args)
    assert d.read_status() == (0, 0)
    assert np.array_equal(B.bits_of(out), expect)
    assert bool((buf[:guard] == 77).all()) and bool((buf[guard + w.numel:] == 77).all())
    return d, out, expect


def _set(sizes, table_log, n_streams, chunk, dtype="bf16", b=4, p0=0.6):
    layers = [W.tiny(seed=s, n=n, bitwidth=b, n_streams=n_streams, chunk_size=chunk, table_log=table_log, p0=p0).layers[0] for s, n in enumerate(sizes)]
    return W.Workload("few", layers, table_log, n_streams, chunk, dtype)


@pytest.mark.parametrize("dtype", ["u8", "f32", "bf16"])
@pytest.mark.parametrize("table_log,N", [(1, 64), (4, 7), (8, 64), (9, 17), (10, 64), (11, 33), (12, 64), (12, 1)])
def test_tables_streams_and_types(orc, table_log, N, dtype):
    sizes = [1, 15, 64 * N + 3, 700, 8 * N]                        # chunks at odd offsets, fewer symbols than streams
    _check(orc, _set(sizes, table_log, N, 1000, dtype, b=1 if table_log == 1 else 4 if table_log >= 5 else 2), planned=table_log % 2 == 0)


# (which kernel each of these goes to is looked at in test_decode_choice.py)
def numbers_of_chunks(n_chunks, table_log):
    return _set([300 * n_chunks - 7], table_log, 64, 300)


NUMBERS = [(n, t, ("few 1" if n <= 256 or t == 12 else "few 2") if n <= 512 else "waves")
           for t in (9, 12) for n in (1, 2, 255, 256, 257, 511, 512, 513, 768, 769, 1024, 1025)]


@pytest.mark.parametrize("n_chunks,table_log,kernel", NUMBERS)
def test_numbers_of_chunks(orc, n_chunks, table_log, kernel):
    _check(orc, numbers_of_chunks(n_chunks, table_log))


# Layers of fewer than eight chunks each, which decode_waves does not take: up to four workgroups per CU
def layers_of_few_chunks(n_layers, chunks, table_log, dtype):
    w = _set([190 * chunks - s % 61 for s in range(n_layers)] + [70000], table_log, 64, 190, dtype)
    w.chunk_sizes = [190] * n_layers + [70000]                      # the last layer: one chunk of several windows
    return w


LAYERS = [(130, 4, 10, "u8", "few 3"), (130, 5, 10, "f32", "few 3"), (130, 5, 10, "bf16", "few 3"), (255, 3, 9, "bf16", "few 3"),
          (192, 4, 9, "u8", "few 4"), (130, 7, 9, "f32", "few 4"), (146, 7, 8, "bf16", "few 4"), (130, 7, 10, "bf16", "few 3"), (60, 5, 12, "bf16", "few 1")]


@pytest.mark.parametrize("n_layers,chunks,table_log,dtype,kernel", LAYERS)
def test_layers_of_few_chunks(orc, n_layers, chunks, table_log, dtype, kernel):
    _check(orc, layers_of_few_chunks(n_layers, chunks, table_log, dtype))


@pytest.mark.parametrize("table_log,sizes,chunk,dtype", [
    (12, [20480], 20480, "bf16"), (12, [12288, 5], 12288, "f32"), (12, [24575] + [64] * 40, 65536, "u8"),
    (12, [150000] + [640] * 60, 200000, "bf16"),                    # a chunk of two windows among short ones
    (10, [400001, 17] + [640] * 200, 500000, "f32"),                # four windows
    (9, [70000] + [128] * 300, 80000, "bf16"),                      # two workgroups per CU, two windows
    (12, [24576, 24577, 24569, 3] + [640] * 60, 65536, "bf16"),     # the longest in one window, the shortest in two
    (11, [32768, 32775, 5, 98304] + [301] * 60, 100000, "f32"),     # a last window of a quarter; windows that LDS bounds
    (10, [200003, 29] + [500] * 300, 200003, "u8"),                 # odd places in the output, two on a CU, windows of 24,000 and a rest
])
def test_long_chunks_among_short_ones(orc, table_log, sizes, chunk, dtype):
    _check(orc, _set(sizes, table_log, 64, chunk, dtype))


def test_a_chunk_whose_words_do_not_fit(orc):
    layers = [W.Layer("dense", (1, 1, 1, 150000), 8, 128, 0.02, np.full(256, 1 / 256), 5)]
    layers += [W.tiny(seed=s, n=640, bitwidth=3, n_streams=64, chunk_size=640, table_log=12, p0=0.8).layers[0] for s in range(100)]
    _check(orc, W.Workload("dense", layers, 12, 64, 150000, "bf16"))


# table_log, short chunks, symbols of the long one, and the kernel (the dispatch is looked at in test_decode_choice.py)
MANY_WORDS = [
    (12, 300, 40000, "few 1"),                                     # 10,000 words: two workgroups per CU would have room for 3,400
    (12, 300, 46400, "few 1"), (11, 300, 22200, "few 2"),          # about the longest the look-ahead kernel holds
    (11, 600, 22200, "few 2"), (10, 600, 22200, "few 3"), (9, 900, 22200, "few 4"),
]


def many_words(table_log, n_short, long):
    layers = [W.Layer("dense", (1, 1, 1, long), 8, 128, 0.02, np.full(256, 1 / 256), 5)]
    layers += [W.tiny(seed=s, n=200, bitwidth=3, n_streams=64, chunk_size=200, table_log=table_log, p0=0.8).layers[0] for s in range(n_short)]
    return W.Workload("dense", layers, table_log, 64, 150000, "bf16")


@pytest.mark.parametrize("table_log,n_short,long,kernel", MANY_WORDS)
def test_a_chunk_of_many_words_among_short_ones(orc, table_log, n_short, long, kernel):
    _check(orc, many_words(table_log, n_short, long))


def _time(call, n=40):
    for _ in range(5):
        call()
    best = float("inf")
    for _ in range(6):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(n):
            call()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) / n)
    return best


# Chunks much longer than the mean, which is what the dispatch knows: beside the look-ahead kernel, forced, the call may not take
# much longer (it takes 0.8 and 1.06 times as long; 6.4 times with words that did not fit LDS, 1.5 and 1.7 where stores
# waited for the walk and the walk for the stores).
@pytest.mark.parametrize("sizes,table_log,p0,dtype", [([2000] * 440 + [65536] * 20, 12, 0.55, "bf16"), ([1000] * 200 + [1 << 20], 12, 0.97, "bf16"),
                                                      ([1000] * 200 + [1 << 20], 12, 0.97, "f32")])
def test_a_long_chunk_among_short_ones_does_not_slow_the_call_down(orc, sizes, table_log, p0, dtype):
    w = _set(sizes, table_log, 64, max(sizes), dtype, p0=p0)
    d = B.to_device(host_from_oracle(oracle_encode(orc, w), w))
    args = B.decode_args(d, B.alloc_out(d))
    here, there = _time(lambda: B.decode_raw(args)), _time(lambda: B.decode_raw(args, variant=B.VARIANT_MERGED))
    assert d.read_status() == (0, 0) and here < 1.3 * there, (here, there)


def test_a_scale_per_channel(orc):
    for clen in (1, 7, 9 * 64, 100000):
        n = 5003
        lay = W.tiny(seed=clen, n=n, bitwidth=5, n_streams=64, chunk_size=2000, table_log=11, p0=0.5).layers[0]
        lay.channel_len = clen
        lay.channel_scales = (0.01 + 0.001 * np.arange(-(-n // clen))).astype(np.float32)
        for dtype in ("bf16", "f32"):
            _check(orc, W.Workload("channels", [lay], 11, 64, 2000, dtype))


def test_corrupt_words_are_reported_and_stay_inside(orc):
    w = _set([8000, 3001], 11, 64, 4000)
    d, out, expect = _check(orc, w)
    rng = np.random.default_rng(3)
    for _ in range(6):
        h = d.host
        bad = h.payload.copy()
        at = rng.integers(0, len(bad), 20)
        bad[at] ^= rng.integers(1, 1 << 32, 20, dtype=np.uint64).astype(np.uint32)
        d.payload.copy_(torch.from_numpy(bad.view(np.uint8)).to("cuda:0"))
        buf = torch.full((w.numel + 8192,), 77, dtype=torch.bfloat16, device="cuda:0")
        d.status.zero_()
        B.decode(d, out=buf[4096:4096 + w.numel])
        assert d.read_status()[0] & (B.ST_BAD_STATE | B.ST_BAD_LENGTH)
        assert bool((buf[:4096] == 77).all()) and bool((buf[4096 + w.numel:] == 77).all())


def test_replayed_from_a_captured_graph(orc):
    w = _set([9000, 777], 10, 64, 3000)
    d, out, expect = _check(orc, w)
    args = B.decode_args(d, out)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        B.decode_raw(args)
    for _ in range(4):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(B.bits_of(out), expect) and d.read_status() == (0, 0)
