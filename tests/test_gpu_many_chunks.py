"""GPU parity of the kernel that decodes a chunk per wavefront (more chunks than the look-ahead kernel decodes at once),
against the oracle bit for bit: shares of a workgroup that begin and end inside layers, layers of few chunks, chunks of one
symbol and of several buffers, chunks with more words than their wavefront's LDS holds, all stream counts, chunks at odd offsets,
scales per channel, a plan that is not needed, and streams that do not end where they should."""
import numpy as np
import pytest
import torch

from paper_2406_06237_amd import binding as B
from paper_2406_06237_amd import workloads as W

from helpers import host_from_oracle, oracle_encode, oracle_expected

pytestmark = pytest.mark.gpu


def _check(orc, w, dtype, at_least=1025):
    c = oracle_encode(orc, w)
    assert c.n_chunks >= at_least and c.n_chunks >= 8 * len(w.layers)
    _, expect = oracle_expected(orc, c, w, dtype)
    d = B.to_device(host_from_oracle(c, w))
    out = B.alloc_out(d, dtype)
    args = B.decode_args(d, out, dtype)
    plan = B.plan_decode(args, d.device)
    for planned in (False, True):
        out.view(torch.uint8).fill_(0xA5)
        B.decode_planned_raw(args, plan, d.device) if planned else B.decode_raw(args, d.device)
        assert d.read_status() == (0, 0)
        bad = np.nonzero(B.bits_of(out)[:w.numel] != expect)[0]
        assert len(bad) == 0, f"{len(bad)} mismatches, first at {bad[:5]}"
    return c, d, expect


@pytest.mark.parametrize("dtype", ["u8", "f32", "bf16"])
@pytest.mark.parametrize("table_log,n_streams,chunk,sizes,p0", [
    (12, 64, 2048, (700001, 3, 1500001, 30000, 2048 * 40), 0.8),     # shares across layers, a layer of one chunk
    (9, 64, 4096, (5000011,), 0.4),
    (5, 33, 100, (99, 60001, 50505), 0.6),                            # small tables and chunks, several to a wavefront
    (12, 64, 16384, (20000003,), 0.85),                               # several buffers a chunk
    (10, 17, 6592, (7000001,), 0.3),
    (11, 1, 1000, (1200001,), 0.7),                                   # one stream, too short to be split
    (8, 64, 1, (1500, 1300), 0.9), (12, 7, 3, (5001,), 0.5),          # chunks of fewer symbols than streams
    (10, 64, 8192, (9000001,), 0.99),                                 # nearly every entry stands for eight symbols
])
def test_many_chunks(orc, dtype, table_log, n_streams, chunk, sizes, p0):
    layers = [W.Layer(f"l{i}", (n,), 4, 8, 0.02 + 0.01 * i, W.peaked_geometric_pmf(16, 8, p0 if i % 2 == 0 else 0.3), 5 + i) for i, n in enumerate(sizes)]
    _check(orc, W.Workload("many", layers, table_log, n_streams, chunk, dtype), dtype)


@pytest.mark.parametrize("n_layers,chunks", [(48, 23), (130, 9), (129, 8)])
def test_many_layers(orc, n_layers, chunks):
    layers = [W.Layer(f"l{i}", (chunks * 1024 - (i * 37) % 256,), 3, 4, 0.01 + 0.001 * i, W.peaked_geometric_pmf(8, 4, 0.5 + 0.003 * i), 5 + i) for i in range(n_layers)]
    _check(orc, W.Workload("layers", layers, 12, 64, 1024, "bf16"), "bf16")


@pytest.mark.parametrize("table_log", [10, 12])
def test_chunks_of_more_words_than_fit(orc, table_log):
    """A few layers of 8 bits a symbol among many of a tenth: shorter buffers beside their words, or words read in place."""
    thin = [W.Layer(f"t{i}", (1200 * 8192,), 4, 8, 0.02, W.peaked_geometric_pmf(16, 8, 0.985), 5 + i) for i in range(1)]
    dense = [W.Layer(f"d{i}", (n,), 8, 128, 0.01, np.ones(256) / 256 if i else W.laplace_pmf(256, 128, 8.0), 50 + i) for i, n in enumerate((20 * 8192, 5 * 8192 + 77))]
    _check(orc, W.Workload("mixed", dense[:1] + thin + dense[1:], table_log, 64, 8192, "bf16"), "bf16")


@pytest.mark.parametrize("channel", [1, 7, 300, 4608])
def test_scales_per_channel(orc, channel):
    rng = np.random.default_rng(channel)
    layers = [W.Layer(f"l{i}", (rows, channel), 4, 8, 0.0, W.laplace_pmf(16, 8, 1.0), 9 + i, channel_len=channel,
                      channel_scales=rng.uniform(0.005, 0.05, rows).astype(np.float32)) for i, rows in enumerate((3, 900000 // channel, 700001 // channel))]
    layers.append(W.Layer("one scale", (50001,), 4, 8, 0.03, W.laplace_pmf(16, 8, 1.0), 19))
    for dtype in ("bf16", "f32"):
        _check(orc, W.Workload("channels", layers, 10, 64, 1024, dtype), dtype)


def test_streams_that_do_not_end_where_they_should(orc):
    """Each broken chunk is reported once, every other one is whole (a wavefront goes on with the next), nothing is written
    outside; words that were never a stream end too."""
    layers = [W.Layer("one", (1100 * 2048,), 4, 8, 0.02, W.laplace_pmf(16, 8, 1.0), 5)]
    c, d, expect = _check(orc, W.Workload("broken", layers, 11, 64, 2048, "bf16"), "bf16")
    n = d.host.numel
    broken = [3, 500, 1099]
    h = d.host.stream_hdr.copy()
    for i in broken:
        h[64 * i + 5] ^= 0x7
    d.stream_hdr.copy_(torch.from_numpy(h.view(np.uint8).copy()))
    chunks = d.host.chunks.copy()
    chunks["layer_id"][700] = 9                                       # no such layer
    chunks["payload_offset"][20] = 1 << 40
    d.chunks.copy_(torch.from_numpy(chunks.view(np.uint8).reshape(-1).copy()))
    buf = torch.full((n + 128,), 0x5A5A, dtype=torch.int16, device="cuda:0")
    out = buf[64:64 + n].view(torch.bfloat16)
    d.status.zero_()
    B.decode_raw(B.decode_args(d, out), d.device)
    st = d.read_status()
    assert st[1] == len(broken) + 2 and st[0] & B.ST_BAD_DESC and st[0] & B.ST_BAD_STATE, st
    got = B.bits_of(out).reshape(1100, 2048)
    whole = [i for i in range(1100) if i not in broken + [700, 20]]
    assert np.array_equal(got[whole], expect.reshape(1100, 2048)[whole])
    assert (got[700] == 0x5A5A).all() and (got[20] == 0x5A5A).all()
    assert bool((buf[:64] == 0x5A5A).all()) and bool((buf[64 + n:] == 0x5A5A).all())
    g = torch.Generator(device="cuda:0").manual_seed(3)
    d.payload.copy_(torch.randint(0, 256, (d.payload.numel(),), dtype=torch.uint8, device="cuda:0", generator=g))
    d.status.zero_()
    B.decode_raw(B.decode_args(d, out), d.device)
    st = d.read_status()
    assert st[0] & (B.ST_BAD_STATE | B.ST_BAD_LENGTH) and st[1] <= 1100
    assert bool((buf[:64] == 0x5A5A).all()) and bool((buf[64 + n:] == 0x5A5A).all())


# ---- descriptors in any order, chunks of any size: shares of equal weight, layer after layer, instead of descriptors in a row
def _in_order(d, order):
    c = d.host.chunks
    if order == "shuffled":
        idx = np.random.default_rng(len(c)).permutation(len(c))
    elif order == "most words first":
        idx = np.argsort(-c["payload_words"].astype(np.int64), kind="stable")
    else:                                                            # the layers' chunks in turn
        idx = np.argsort(np.concatenate([np.arange(k) for k in np.bincount(c["layer_id"])]), kind="stable")
    d.chunks.copy_(torch.from_numpy(np.ascontiguousarray(c[idx]).view(np.uint8).reshape(-1).copy()))


def _check_order(orc, w, dtype, order):
    """Bit for bit; then, with a stream's length wrong in every chunk, every chunk is reported once: none is left out or decoded twice."""
    c = oracle_encode(orc, w)
    assert c.n_chunks >= 1025 and c.n_chunks >= 8 * len(w.layers)
    _, expect = oracle_expected(orc, c, w, dtype)
    d = B.to_device(host_from_oracle(c, w))
    _in_order(d, order)
    out = B.alloc_out(d, dtype)
    args = B.decode_args(d, out, dtype)
    out.view(torch.uint8).fill_(0xA5)
    B.decode_raw(args, d.device)
    assert d.read_status() == (0, 0)
    bad = np.nonzero(B.bits_of(out)[:w.numel] != expect)[0]
    assert len(bad) == 0, f"{len(bad)} mismatches, first at {bad[:5]}"
    h = d.host.stream_hdr.copy()
    h[::w.n_streams] += 1 << 16
    d.stream_hdr.copy_(torch.from_numpy(h.view(np.uint8).copy()))
    B.decode_raw(args, d.device)
    st = d.read_status()
    assert st[1] == c.n_chunks and st[0] & B.ST_BAD_DESC, st[:2]


@pytest.mark.parametrize("order", ["shuffled", "most words first", "in turn"])
@pytest.mark.parametrize("table_log,n_streams,chunk,n_layers,chunks,p0", [
    (12, 64, 1024, 48, 23, 0.6),              # few chunks a workgroup
    (9, 17, 100, 7, 1290, 0.5),               # more than are sorted at once
    (12, 64, 4096, 130, 9, 0.8), (10, 33, 1000, 2, 600, 0.7), (11, 1, 500, 48, 30, 0.6),
])
def test_descriptors_in_any_order(orc, order, table_log, n_streams, chunk, n_layers, chunks, p0):
    layers = [W.Layer(f"l{i}", ((chunks - i % 3) * chunk - (i * 37) % 99,), 4, 8, 0.01 + 0.001 * i, W.peaked_geometric_pmf(16, 8, p0 + 0.39 * (i % 7) / 7), 5 + i)
              for i in range(n_layers)]
    w = W.Workload("order", layers, table_log, n_streams, chunk, "bf16")
    _check_order(orc, w, ("bf16", "u8", "f32")[chunk % 3], order)


@pytest.mark.parametrize("order", ["shuffled", "most words first", "in turn"])
@pytest.mark.parametrize("table_log,n_streams,chunk", [(12, 64, 8192), (10, 16, 16384), (12, 8, 5000)])
def test_long_chunks_among_short_ones(orc, order, table_log, n_streams, chunk):
    """8 bits a symbol beside a tenth: the long ones take a turn of their own, several at a time."""
    pmfs = [W.peaked_geometric_pmf(16, 8, 0.985)] * 2 + [np.ones(256) / 256, W.laplace_pmf(256, 128, 7.0)] + [W.peaked_geometric_pmf(16, 8, 0.97)] * 2
    sizes = [300 * chunk, 250 * chunk - 5, 40 * chunk, 30 * chunk - 77, 400 * chunk, 100 * chunk]
    layers = [W.Layer(f"l{i}", (n,), 8, 8, 0.02, pmf, 5 + i) for i, (n, pmf) in enumerate(zip(sizes, pmfs))]
    _check_order(orc, W.Workload("long", layers, table_log, n_streams, chunk, "bf16"), "bf16", order)


def test_chunks_of_more_words_than_a_workgroup_holds(orc):
    """32,768 words: one symbol at a time from memory, as in every kernel whose window they exceed; 16,384: alone in LDS."""
    chunk = 131072
    layers = [W.Layer("thin", (1030 * chunk,), 8, 8, 0.02, W.peaked_geometric_pmf(16, 8, 0.998), 5), W.Layer("long", (2 * chunk,), 8, 8, 0.02, np.ones(256) / 256, 6),
              W.Layer("half", (2 * chunk,), 8, 8, 0.02, W.laplace_pmf(16, 8, 4.0), 7)]
    _check_order(orc, W.Workload("window", layers, 12, 64, chunk, "u8"), "u8", "most words first")


@pytest.mark.parametrize("singles,rest", [(150, 1200), (11, 1100)])
def test_layers_of_one_chunk_in_a_row(orc, singles, rest):
    sizes = [rest // 2 * 1024] + [1024 - i % 7 for i in range(singles)] + [rest // 2 * 1024 - 3]
    layers = [W.Layer(f"l{i}", (n,), 4, 8, 0.01 + 0.001 * i, W.peaked_geometric_pmf(16, 8, 0.5 + 0.003 * (i % 99)), 5 + i) for i, n in enumerate(sizes)]
    _check(orc, W.Workload("singles", layers, 12, 64, 1024, "bf16"), "bf16")


def test_a_share_of_several_windows(orc):
    """8,200 single streams of 1,000 words before 150,000 of ten: a share of the first descriptors sorted at once is longer than its list."""
    pmf = np.ones(256) / 256
    w = W.Workload("windows", [W.Layer("long", (8200 * 4000,), 8, 128, 0.02, pmf, 5), W.Layer("short", (150000 * 40,), 8, 128, 0.03, pmf, 6)], 9, 1, 4000, "u8")
    w.chunk_sizes = [4000, 40]
    _check_order(orc, w, "u8", "most words first")
