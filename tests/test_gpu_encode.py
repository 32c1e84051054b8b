"""GPU parity of the device packer: anszp_pack_layer_device through the C ABI must write, word for word,
the container the ORACLE's encoder writes for the same symbols and frequencies."""
import numpy as np
import pytest
import torch

from paper_2406_06237_amd import binding as B
from paper_2406_06237_amd import workloads as W

pytestmark = pytest.mark.gpu


def _pack(sym, freqs, R, N, chunk, **kw):
    s = torch.from_numpy(np.ascontiguousarray(sym, dtype=np.uint8)).to("cuda:0")
    f = torch.from_numpy(np.ascontiguousarray(freqs, dtype=np.uint32).view(np.int32)).to("cuda:0")
    chunks, hdr, payload, used, status = B.pack_layer_device(s, f, R, N, chunk, **kw)
    torch.cuda.synchronize()
    st = status.cpu().numpy().view(np.uint32)
    return (chunks.cpu().numpy().view(B.CHUNK_DTYPE), hdr.cpu().numpy().view(np.uint32), payload.cpu().numpy().view(np.uint32),
            int(used.item()), (int(st[0]), int(st[1])))


def _compare(orc, sym, R, N, chunk):
    c = orc.encode_layers([sym], R, N, chunk)
    chunks, hdr, payload, used, status = _pack(sym, c.freqs[0], R, N, chunk)
    assert status == (0, 0)
    assert used == len(c.payload)
    nc = c.n_chunks
    assert np.array_equal(chunks["layer_id"][:nc], c.chunk_layer)
    assert np.array_equal(chunks["n_symbols"][:nc], c.chunk_nsym)
    assert np.array_equal(chunks["out_offset"][:nc], c.chunk_out_off)
    assert np.array_equal(chunks["payload_offset"][:nc], c.chunk_payload_off)
    assert np.array_equal(chunks["payload_words"][:nc], c.chunk_payload_words)
    assert np.array_equal(chunks["stream_offset"][:nc], c.chunk_stream_off)
    assert np.array_equal(hdr[:nc * N], c.stream_hdr)
    assert np.array_equal(payload[:used], c.payload)
    assert np.all(payload[used:] == 0xFFFFFFFF)                  # nothing written beyond what is reported


@pytest.mark.parametrize("N,chunk,n,R,b,p0", [
    (64, 2048, 5000, 10, 4, 0.8), (64, 65536, 65536 + 1000, 12, 8, 0.7), (32, 16384, 40000, 11, 3, 0.6),
    (1, 3000, 7001, 10, 4, 0.5), (7, 100, 999, 9, 2, 0.9), (64, 4096, 40, 8, 5, 0.75),
    (64, 1024, 3 * 1024, 12, 1, 0.95), (33, 555, 5555, 6, 6, 0.3), (64, 128, 1, 5, 4, 0.8),
])
def test_ragged_geometries(orc, N, chunk, n, R, b, p0):
    w = W.tiny(seed=n, n=n, bitwidth=b, n_streams=N, chunk_size=chunk, table_log=R, p0=p0)
    _compare(orc, w.symbols()[0], R, N, chunk)


def test_layers_of_the_benchmark_sets(orc):
    w = W.config1()
    _compare(orc, w.symbols()[0], w.table_log, w.n_streams, w.chunk_size)
    w = W.config3()
    for i in (0, 13, 44):
        _compare(orc, w.layers[i].symbols(), w.table_log, w.n_streams, w.chunk_size)


def test_single_symbol_and_flat_distributions(orc):
    _compare(orc, np.full(10000, 4, dtype=np.uint8), 12, 64, 4096)
    _compare(orc, np.random.default_rng(1).integers(0, 256, 50000).astype(np.uint8), 12, 64, 8192)


def test_decoder_reads_what_the_packer_wrote(orc):
    w = W.tiny(seed=5, n=150000, bitwidth=4, n_streams=64, chunk_size=32768, table_log=12, p0=0.8)
    sym = w.symbols()[0]
    c = orc.encode_layers([sym], 12, 64, 32768)
    s = torch.from_numpy(sym).to("cuda:0")
    f = torch.from_numpy(c.freqs[0].astype(np.uint32).view(np.int32)).to("cuda:0")
    chunks, hdr, payload, used, status = B.pack_layer_device(s, f, 12, 64, 32768)
    tables = B.build_tables(c.freqs, 12, "cuda:0")
    lay = w.layers[0]
    layers = np.zeros(1, dtype=B.LAYER_DTYPE)
    layers[0] = (lay.scale, lay.zero_point, lay.bitwidth, 0, 0, 0)
    out = torch.empty(len(sym), dtype=torch.uint8, device="cuda:0")
    st = torch.zeros(2, dtype=torch.int32, device="cuda:0")
    a = B.DecodeArgs()
    a.tables = tables.data_ptr(); a.n_tables = 1; a.table_log = 12; a.n_streams = 64; a.out_dtype = B.OUT_U8
    a.chunks = chunks.data_ptr(); a.n_chunks = c.n_chunks
    a.stream_hdr = hdr.data_ptr(); a.n_stream_hdr = c.n_chunks * 64
    a.payload = payload.data_ptr(); a.payload_words = int(used.item())
    ldev = torch.from_numpy(layers.view(np.uint8)).to("cuda:0")
    a.layers = ldev.data_ptr(); a.scales = 0; a.n_scales = 0
    a.out = out.data_ptr(); a.out_elems = len(sym); a.status = st.data_ptr()
    B.decode_raw(a, "cuda:0")
    torch.cuda.synchronize()
    assert tuple(st.cpu().numpy()) == (0, 0)
    assert np.array_equal(out.cpu().numpy(), sym)


def test_errors_are_reported(orc):
    sym = np.array([0, 1, 2, 1, 0, 1] * 100, dtype=np.uint8)
    f = np.zeros(256, dtype=np.uint32); f[0], f[1] = 512, 512          # symbol 2 has no frequency
    assert _pack(sym, f, 10, 8, 64)[4][0] & B.ST_BAD_SYMBOL
    f[2] = 5                                                            # does not sum to 1024
    chunks, hdr, payload, used, status = _pack(sym, f, 10, 8, 64)
    assert status[0] & B.ST_BAD_FREQ and np.all(payload == 0xFFFFFFFF)
    c = orc.encode_layers([sym], 10, 8, 64)
    chunks, hdr, payload, used, status = _pack(sym, c.freqs[0], 10, 8, 64, payload_cap_words=8)
    assert status[0] & B.ST_NO_SPACE and used == len(c.payload) and np.all(payload[8:] == 0xFFFFFFFF)


# ---- a whole set in three launches (anszp_pack_layers_device)
def _pack_set(w, orc_container):
    syms = w.symbols()
    s = torch.from_numpy(np.concatenate(syms)).to("cuda:0")
    f = torch.from_numpy(np.ascontiguousarray(orc_container.freqs, dtype=np.uint32).view(np.int32)).to("cuda:0")
    sizes = getattr(w, "chunk_sizes", None) or w.chunk_size
    chunks, hdr, payload, used, status = B.pack_layers_device(s, [len(x) for x in syms], f, w.table_log, w.n_streams, sizes)
    torch.cuda.synchronize()
    st = status.cpu().numpy().view(np.uint32)
    return (chunks.cpu().numpy().view(B.CHUNK_DTYPE), hdr.cpu().numpy().view(np.uint32), payload.cpu().numpy().view(np.uint32),
            int(used.item()), (int(st[0]), int(st[1])))


@pytest.mark.parametrize("name", ["config2", "config3", "channel_grouped", "odd_bins", "mixed"])
def test_whole_sets_in_one_call_equal_the_oracles_container(orc, name):
    if name == "mixed":                                            # layers of 1 to 70,001 symbols, 48 streams
        layers = [W.tiny(seed=s, n=n, bitwidth=b, n_streams=48, chunk_size=3000, table_log=10, p0=0.7).layers[0]
                  for s, (n, b) in enumerate([(1, 2), (70001, 4), (2999, 1), (3000, 8), (3001, 3), (47, 5)])]
        w = W.Workload("mixed", layers, 10, 48, 3000, "bf16")
    else:
        w = {"config2": W.config2, "config3": W.config3, "channel_grouped": W.channel_grouped, "odd_bins": W.resnet50_odd_bins}[name]()
    from helpers import oracle_encode
    c = oracle_encode(orc, w)
    chunks, hdr, payload, used, status = _pack_set(w, c)
    assert status == (0, 0)
    assert used == len(c.payload)
    nc, N = c.n_chunks, w.n_streams
    for field, want in (("layer_id", c.chunk_layer), ("n_symbols", c.chunk_nsym), ("out_offset", c.chunk_out_off),
                        ("payload_offset", c.chunk_payload_off), ("payload_words", c.chunk_payload_words),
                        ("stream_offset", c.chunk_stream_off)):
        assert np.array_equal(chunks[field][:nc], want), field
    assert np.array_equal(hdr[:nc * N], c.stream_hdr)
    assert np.array_equal(payload[:used], c.payload)
    assert np.all(payload[used:] == 0xFFFFFFFF)


def _same(c, w, out):
    chunks, hdr, payload, used, status = (t.cpu().numpy() for t in out)
    nc = c.n_chunks
    assert tuple(status) == (0, 0) and int(used[0]) == len(c.payload)
    assert np.array_equal(payload.view(np.uint32)[:len(c.payload)], c.payload) and np.array_equal(hdr.view(np.uint32)[:nc * w.n_streams], c.stream_hdr)
    assert np.array_equal(chunks.view(B.CHUNK_DTYPE)["payload_offset"][:nc], c.chunk_payload_off)
    assert np.array_equal(chunks.view(B.CHUNK_DTYPE)["out_offset"][:nc], c.chunk_out_off)


def test_a_whole_set_is_packed_in_order_on_its_stream(orc):
    """The call does not wait: another stream that waits for an event behind it reads the whole container, and what stands behind
    the call on its own stream may overwrite the symbols."""
    w = W.config2()
    from helpers import oracle_encode
    c = oracle_encode(orc, w)
    syms = w.symbols()
    host = torch.from_numpy(np.concatenate(syms)).pin_memory()
    f = torch.from_numpy(np.ascontiguousarray(c.freqs, dtype=np.uint32).view(np.int32)).to("cuda:0")
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    for _ in range(5):
        with torch.cuda.stream(a):
            s = host.to("cuda:0", non_blocking=True)
            out = B.pack_layers_device(s, [len(x) for x in syms], f, w.table_log, w.n_streams, w.chunk_size)
            done = torch.cuda.Event()
            done.record()
            s.zero_()
        with torch.cuda.stream(b):
            b.wait_event(done)
            copies = [t.clone() for t in out]
        b.synchronize()
        _same(c, w, copies)
    torch.cuda.synchronize()


def test_a_whole_set_is_refused_under_capture(orc):
    w = W.config2()
    from helpers import oracle_encode
    c = oracle_encode(orc, w)
    s = torch.from_numpy(np.concatenate(w.symbols())).to("cuda:0")
    f = torch.from_numpy(np.ascontiguousarray(c.freqs, dtype=np.uint32).view(np.int32)).to("cuda:0")
    sizes = [len(x) for x in w.symbols()]
    out = B.pack_layers_device(s, sizes, f, w.table_log, w.n_streams, w.chunk_size)
    torch.cuda.synchronize()
    with torch.cuda.graph(torch.cuda.CUDAGraph()):
        with pytest.raises(RuntimeError, match="captur"):
            B.pack_layers_device(s, sizes, f, w.table_log, w.n_streams, w.chunk_size, out=out)
    out = B.pack_layers_device(s, sizes, f, w.table_log, w.n_streams, w.chunk_size)
    torch.cuda.synchronize()
    _same(c, w, out)


def test_packing_on_three_streams_beside_each_other(orc):
    """Workgroups of several packs share the chip: each waits for lower-numbered ones of its own, and every container is whole."""
    from helpers import oracle_encode
    jobs = []
    for i, w in enumerate((W.config2(), W.config3(), W.tiny(seed=5, n=700001, n_streams=48, chunk_size=1400, table_log=11))):
        c = oracle_encode(orc, w)
        s = torch.from_numpy(np.concatenate(w.symbols())).to("cuda:0")
        f = torch.from_numpy(np.ascontiguousarray(c.freqs, dtype=np.uint32).view(np.int32)).to("cuda:0")
        jobs.append((w, c, s, f, torch.cuda.Stream()))
    torch.cuda.synchronize()
    for _ in range(4):
        outs = []
        for w, c, s, f, stream in jobs:
            with torch.cuda.stream(stream):
                outs.append(B.pack_layers_device(s, [len(x) for x in w.symbols()], f, w.table_log, w.n_streams, w.chunk_size))
        torch.cuda.synchronize()
        for (w, c, *_), out in zip(jobs, outs):
            _same(c, w, out)


def test_whole_set_error_bits_and_rate(orc):
    w = W.config3()
    syms = w.symbols()
    from helpers import oracle_encode
    c = oracle_encode(orc, w)
    s = torch.from_numpy(np.concatenate(syms)).to("cuda:0")
    f = torch.from_numpy(np.ascontiguousarray(c.freqs, dtype=np.uint32).view(np.int32)).to("cuda:0")
    sizes = [len(x) for x in syms]
    out = B.pack_layers_device(s, sizes, f, w.table_log, w.n_streams, w.chunk_size)
    # the rate of the whole set, outputs reused (printed with -s; the host packer does 0.3 Gsymbols/s on one thread)
    import time
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(5):
        B.pack_layers_device(s, sizes, f, w.table_log, w.n_streams, w.chunk_size, out=out)
    torch.cuda.synchronize()
    dt = (time.perf_counter() - t0) / 5
    print(f"anszp_pack_layers_device: {w.numel} symbols in {dt * 1e3:.2f} ms = {w.numel / dt / 1e9:.2f} Gsymbols/s")
    assert np.array_equal(out[2].cpu().numpy().view(np.uint32)[:len(c.payload)], c.payload)
    assert w.numel / dt / 1e9 > 3.0                                  # ten host threads' worth
    # a frequency row that does not sum to L, a symbol without a frequency, a payload buffer that is too small
    bad = f.clone()
    bad[3, 0] += 1
    st = B.pack_layers_device(s, sizes, bad, w.table_log, w.n_streams, w.chunk_size)[4].cpu().numpy().view(np.uint32)
    assert st[0] & B.ST_BAD_FREQ
    s2 = s.clone()
    unused = int(np.nonzero(c.freqs[0] == 0)[0][0])
    s2[5] = unused
    st = B.pack_layers_device(s2, sizes, f, w.table_log, w.n_streams, w.chunk_size)[4].cpu().numpy().view(np.uint32)
    assert st[0] & B.ST_BAD_SYMBOL
    small = B.pack_layers_device(s, sizes, f, w.table_log, w.n_streams, w.chunk_size, payload_cap_words=len(c.payload) // 2)
    st = small[4].cpu().numpy().view(np.uint32)
    assert st[0] & B.ST_NO_SPACE and int(small[3].item()) == len(c.payload)
    assert np.all(small[2].cpu().numpy().view(np.uint32)[len(c.payload) // 2:] == 0xFFFFFFFF)


# A walk takes a stream's symbols in batches of sixteen, the first of them short; a workgroup takes several chunks, of
# several layers, once there are more than 512.  Whole words are compared: no tolerance.
@pytest.mark.parametrize("rows", [1, 2, 15, 16, 17, 31, 32, 33, 47, 48, 49, 64, 65])
def test_stream_lengths_around_the_walks_batches(orc, rows):
    for N, tail in ((64, 0), (64, 1), (64, 63), (5, 2), (1, 0)):      # tail: symbols beyond whole rows, in the last chunk
        n = 2 * rows * N + (rows - 1) * N + tail
        _compare(orc, W.tiny(seed=n, n=n, bitwidth=5, table_log=12, p0=0.5).symbols()[0], 12, N, rows * N)


@pytest.mark.parametrize("n_layers,n,chunk", [(40, 3001, 192), (3, 65 * 1500, 65), (700, 130, 64)])
def test_workgroups_of_several_chunks_and_layers(orc, n_layers, n, chunk):
    layers = [W.tiny(seed=s, n=n - s % 7, bitwidth=2 + s % 7, n_streams=64, chunk_size=chunk, table_log=9, p0=0.4 + 0.01 * (s % 50)).layers[0]
              for s in range(n_layers)]
    w = W.Workload("many", layers, 9, 64, chunk, "bf16")
    from helpers import oracle_encode
    c = oracle_encode(orc, w)
    chunks, hdr, payload, used, status = _pack_set(w, c)
    assert status == (0, 0) and used == len(c.payload) and c.n_chunks > 512
    assert np.array_equal(chunks["out_offset"][:c.n_chunks], c.chunk_out_off) and np.array_equal(chunks["payload_offset"][:c.n_chunks], c.chunk_payload_off)
    assert np.array_equal(hdr[:c.n_chunks * 64], c.stream_hdr) and np.array_equal(payload[:used], c.payload)


def test_descriptors_and_headers_are_complete_where_the_payload_has_no_room(orc):
    sym = W.tiny(n=20000, bitwidth=6, table_log=12, p0=0.4).symbols()[0]
    c = orc.encode_layers([sym], 12, 64, 4096)
    chunks, hdr, payload, used, status = _pack(sym, c.freqs[0], 12, 64, 4096, payload_cap_words=1500)
    assert status[0] == B.ST_NO_SPACE and used == len(c.payload) and np.all(payload[1500:] == 0xFFFFFFFF)
    assert np.array_equal(chunks["out_offset"][:c.n_chunks], c.chunk_out_off) and np.array_equal(hdr[:c.n_chunks * 64], c.stream_hdr)


# More chunks than two workgroups per CU have wavefronts: a wavefront then takes several chunks of a run, one after the other.
@pytest.mark.parametrize("n_chunks,per,N", [(4097, 64, 64), (5003, 130, 64), (20000, 33, 7), (70001, 3, 1)])
def test_more_chunks_than_wavefronts(orc, n_chunks, per, N):
    n = n_chunks * per - (per - 1)                                 # the last chunk has one symbol
    _compare(orc, W.tiny(seed=n, n=n, bitwidth=4, table_log=9, p0=0.6).symbols()[0], 9, N, per)


def test_many_layers_of_more_chunks_than_wavefronts(orc):
    layers = [W.tiny(seed=s, n=1700 + 31 * s, bitwidth=2 + s % 5, n_streams=16, chunk_size=32, table_log=8, p0=0.5).layers[0] for s in range(90)]
    w = W.Workload("many", layers, 8, 16, 32, "bf16")
    from helpers import oracle_encode
    c = oracle_encode(orc, w)
    chunks, hdr, payload, used, status = _pack_set(w, c)
    assert status == (0, 0) and used == len(c.payload) and c.n_chunks > 8 * 512
    assert np.array_equal(chunks["out_offset"][:c.n_chunks], c.chunk_out_off) and np.array_equal(chunks["payload_offset"][:c.n_chunks], c.chunk_payload_off)
    assert np.array_equal(hdr[:c.n_chunks * 16], c.stream_hdr) and np.array_equal(payload[:used], c.payload)


def test_more_chunks_than_a_grid_of_workgroups_of_eight_could_hold(orc):
    """2^26 chunks and a few: eight per workgroup of 512 would be more than 2^32 work-items.  Chunks of two symbols in one
    stream, so that the headers and words the oracle gives the 64 pairs are those of all chunks."""
    n, R = (1 << 26) + 5, 6
    freqs = np.zeros(256, dtype=np.uint32)
    freqs[:8] = (5, 3, 9, 7, 11, 13, 6, 10)
    pairs = np.stack([np.arange(64) // 8, np.arange(64) % 8], axis=1).astype(np.uint8)
    c = orc.encode_layers([pairs.reshape(-1)], R, 1, 2, freqs=[freqs])
    assert len(c.payload) == 4 * 64 and np.all(c.chunk_payload_words == 1)
    g = torch.Generator(device="cuda:0")
    g.manual_seed(3)
    sym = torch.randint(0, 8, (2 * n,), generator=g, device="cuda:0", dtype=torch.uint8)
    chunks, hdr, payload, used, status = B.pack_layer_device(sym, torch.from_numpy(freqs.view(np.int32)).to("cuda:0"), R, 1, 2)
    torch.cuda.synchronize()
    assert status.tolist() == [0, 0] and int(used.item()) == 4 * n
    pair = sym[0::2].long() * 8 + sym[1::2].long()
    of_pair = lambda a: torch.from_numpy(np.ascontiguousarray(a).view(np.int32)).to("cuda:0")[pair]
    assert torch.equal(hdr[:n], of_pair(c.stream_hdr))
    words = payload[:4 * n].view(n, 4)
    assert torch.equal(words[:, 0], of_pair(c.payload[::4])) and not bool(words[:, 1:].any())
    rows, i = chunks.view(n, B.CHUNK_DTYPE.itemsize), torch.arange(n, device="cuda:0")
    for field, want, dtype in (("out_offset", 2 * i, torch.int64), ("payload_offset", 4 * i, torch.int64), ("stream_offset", i.int(), torch.int32),
                               ("n_symbols", torch.full_like(i, 2).int(), torch.int32), ("payload_words", torch.ones_like(i).int(), torch.int32)):
        begin = B.CHUNK_DTYPE.fields[field][1]
        assert torch.equal(rows[:, begin:begin + want.element_size()].contiguous().view(dtype)[:, 0], want), field


def test_a_layer_without_symbols_still_has_its_frequencies_checked():
    f = np.zeros(256, dtype=np.uint32)
    f[3], f[255] = 1000, 24
    empty = np.zeros(0, dtype=np.uint8)
    chunks, hdr, payload, used, status = _pack(empty, f, 10, 64, 4096)
    assert status == (0, 0) and used == 0 and np.all(payload == 0xFFFFFFFF)
    for at, v in ((255, 25), (3, 0), (7, 0xFFFFFFFF)):             # one too many, too few, a sum that wraps around
        g = f.copy()
        g[at] = v
        chunks, hdr, payload, used, status = _pack(empty, g, 10, 64, 4096)
        assert status == (B.ST_BAD_FREQ, 1) and used == 0 and np.all(payload == 0xFFFFFFFF)


@pytest.mark.parametrize("polls", [1, 2])
def test_chunks_whose_place_is_not_known_in_time_are_written_all_the_same(orc, polls):
    """Workgroups wait for the word counts of the chunks before theirs; with the bound lowered from the host most give up, and
    where all streams fit LDS (64 rows of at most 11 bits do) the last workgroup to be done writes those chunks."""
    w = W.tiny(seed=11, n=300 * 4096 + 77, bitwidth=5, n_streams=64, chunk_size=4096, table_log=11, p0=0.6)
    try:
        B.lib().anszp_test_set_spin_limit(polls)
        _compare(orc, w.symbols()[0], 11, 64, 4096)
    finally:
        B.lib().anszp_test_set_spin_limit(0)
    _compare(orc, w.symbols()[0], 11, 64, 4096)


@pytest.mark.parametrize("R,N,chunk,n", [(12, 64, 65536, 200000), (8, 64, 36000, 100000), (12, 5, 3000, 40000), (10, 1, 4400, 30000), (9, 1, 200000, 190001)])
def test_streams_longer_than_their_place_in_lds(orc, R, N, chunk, n):
    """Up to 8 bits a symbol: chunks with a stream of more words than LDS holds, beside some that fit, are written by the
    launch behind; 4,400 symbols of one bit are just such a stream, and of half of them not."""
    rng = np.random.default_rng(n)
    dense = rng.integers(0, 256 if R >= 8 else 16, n).astype(np.uint8)
    _compare(orc, dense, R, N, chunk)
    two = rng.integers(0, 2, n).astype(np.uint8)
    two[: n // 3] = 1
    _compare(orc, two, R, N, chunk)
    thin = np.where(rng.random(n) < 0.97, 1, two).astype(np.uint8)
    _compare(orc, np.concatenate([thin, dense, two]), R, N, chunk)


# ---- tables worked out by the launch before the packer (anszp_pack_set_device, behind every call above): occurrences are counted
# against each symbol up to 128 symbols and sorted beyond; 512 of them a workgroup; 64 jobs a launch.
@pytest.mark.parametrize("symbols", [1, 2, 3, 4, 5, 63, 127, 128, 129, 256])
def test_tables_of_any_alphabet(orc, symbols):
    rng = np.random.default_rng(symbols)
    for R in (1, 3, 8, 9, 10, 12):
        if symbols > 1 << R:
            continue
        names = np.sort(rng.choice(256, symbols, replace=False)).astype(np.uint8)
        for weights in (np.ones(symbols), rng.random(symbols) ** 4 + 1e-4):
            sym = np.concatenate([names, rng.choice(names, 3000, p=weights / weights.sum())]).astype(np.uint8)
            _compare(orc, sym, R, 17, 700)


@pytest.mark.parametrize("n_layers", [1, 2, 63, 64, 65, 130])
def test_jobs_by_the_launches_arguments(orc, n_layers):
    layers = [W.tiny(seed=s, n=300 + 17 * s % 500, bitwidth=1 + s % 8, n_streams=32, chunk_size=256, table_log=9, p0=0.6).layers[0] for s in range(n_layers)]
    w = W.Workload("many", layers, 9, 32, 256, "bf16")
    from helpers import oracle_encode
    c = oracle_encode(orc, w)
    chunks, hdr, payload, used, status = _pack_set(w, c)
    assert status == (0, 0) and used == len(c.payload)
    assert np.array_equal(chunks["out_offset"], c.chunk_out_off) and np.array_equal(chunks["payload_offset"], c.chunk_payload_off)
    assert np.array_equal(hdr, c.stream_hdr) and np.array_equal(payload[:used], c.payload) and np.all(payload[used:] == 0xFFFFFFFF)


def _pack_layer_without_scratch(sym, freqs, R, N, chunk, cap, layer_id=0, out_offset=0, payload_word_offset=0, stream_offset=0):
    """anszp_pack_layer_device into cleared results; sym, freqs on the GPU."""
    nc = -(-sym.numel() // chunk)
    out = (torch.zeros(nc * B.CHUNK_DTYPE.itemsize, dtype=torch.uint8, device="cuda:0"), torch.zeros(nc * N, dtype=torch.int32, device="cuda:0"),
           torch.full((cap,), -1, dtype=torch.int32, device="cuda:0"), torch.zeros(1, dtype=torch.int64, device="cuda:0"), torch.zeros(2, dtype=torch.int32, device="cuda:0"))
    assert B.lib().anszp_pack_layer_device(sym.data_ptr(), sym.numel(), freqs.data_ptr(), R, N, chunk, layer_id, out_offset, payload_word_offset, stream_offset,
                                           out[0].data_ptr(), out[1].data_ptr(), out[2].data_ptr(), cap, out[3].data_ptr(), out[4].data_ptr(),
                                           torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    return out


def _pack_without_scratch(w, c):
    """anszp_pack_layers_device: nothing but the results."""
    syms = w.symbols()
    s = torch.from_numpy(np.concatenate(syms)).to("cuda:0")
    f = torch.from_numpy(np.ascontiguousarray(c.freqs, dtype=np.uint32).view(np.int32)).to("cuda:0")
    jobs = torch.from_numpy(B.pack_jobs([len(x) for x in syms], [w.chunk_size] * len(syms)).view(np.uint8)).to("cuda:0")
    nc, cap = c.n_chunks, len(c.payload) + 100
    chunks = torch.zeros(nc * B.CHUNK_DTYPE.itemsize, dtype=torch.uint8, device="cuda:0")
    hdr = torch.zeros(nc * w.n_streams, dtype=torch.int32, device="cuda:0")
    payload = torch.full((cap,), -1, dtype=torch.int32, device="cuda:0")
    used, status = torch.zeros(1, dtype=torch.int64, device="cuda:0"), torch.zeros(2, dtype=torch.int32, device="cuda:0")
    assert B.lib().anszp_pack_layers_device(s.data_ptr(), jobs.data_ptr(), len(syms), nc, f.data_ptr(), w.table_log, w.n_streams, chunks.data_ptr(),
                                            hdr.data_ptr(), payload.data_ptr(), cap, used.data_ptr(), status.data_ptr(),
                                            torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    return chunks, hdr, payload, used, status


@pytest.mark.parametrize("chunk,N", [(5000, 64), (300, 17)])             # few chunks, and more than two per CU
def test_the_entry_points_without_scratch_memory(orc, chunk, N):
    from helpers import oracle_encode
    layers = [W.tiny(seed=s, n=40000 + 17 * s, bitwidth=2 + s, n_streams=N, chunk_size=chunk, table_log=11, p0=0.6).layers[0] for s in range(6)]
    w = W.Workload("raw", layers, 11, N, chunk, "bf16")
    c = oracle_encode(orc, w)
    _same(c, w, _pack_without_scratch(w, c))
    sym, f = w.symbols()[1], torch.from_numpy(c.freqs[1].astype(np.uint32).view(np.int32)).to("cuda:0")
    s = torch.from_numpy(sym).to("cuda:0")
    chunks, hdr, payload, used, status = B.pack_layer_device(s, f, 11, N, chunk, 3, 64, 8, 5)
    again = _pack_layer_without_scratch(s, f, 11, N, chunk, payload.numel(), 3, 64, 8, 5)
    for a, b in zip((chunks, hdr, payload, used, status), again):
        assert torch.equal(a, b)


def test_many_tables_of_many_symbols_are_worked_out_by_the_whole_chip():
    """300 layers whose tables are sorted (more than 128 symbols), a few symbols each: beside the entry point where every workgroup
    sorts for itself and nothing is allocated or cleared, the call may not take much longer (it takes 1.13 times as long; 3.0 with all sorts on one die)."""
    n, rng = 300, np.random.default_rng(4)
    counts = np.full(256, 4000)
    counts[0] += 1000000
    f = torch.from_numpy(np.stack([B.normalize_freqs(counts, 12)] * n).astype(np.int32)).to("cuda:0")
    s = torch.from_numpy(rng.choice(256, 300 * n, p=counts / counts.sum()).astype(np.uint8)).to("cuda:0")
    jobs = torch.from_numpy(B.pack_jobs([300] * n, [4096] * n).view(np.uint8)).to("cuda:0")
    chunks, hdr, payload, used, status = B.pack_layers_device(s, [300] * n, f, 12, 64, 4096)
    again = [torch.zeros_like(chunks), torch.zeros_like(hdr), torch.full_like(payload, -1), torch.zeros_like(used), torch.zeros_like(status)]
    args = [t.data_ptr() for t in again]

    def without_scratch():
        assert B.lib().anszp_pack_layers_device(s.data_ptr(), jobs.data_ptr(), n, n, f.data_ptr(), 12, 64, args[0], args[1], args[2], payload.numel(), args[3], args[4],
                                                torch.cuda.current_stream().cuda_stream) == 0

    def time(call):
        best = float("inf")
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                call()
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b) / 20)
        return best

    there, here = time(without_scratch), time(lambda: B.pack_layers_device(s, [300] * n, f, 12, 64, 4096))
    for a, b in zip((chunks, hdr, payload, used, status), again):
        assert torch.equal(a, b)
    assert here < 1.8 * there, (here, there)


# ---- Given-up waits where some stream may not fit LDS, or there is no scratch memory: the launch behind (encode_rest) writes the chunks
# that were given up, those that fitted LDS among them, and those with a stream that did not fit.
def _long_streams():
    """1,024 rows a chunk at 2^12 states: mostly dominant layers, whose streams fit, around a dense one, whose streams do not."""
    dense = W.Layer("dense", (1, 1, 1, 65536 + 3000), 8, 128, 0.02, np.full(256, 1 / 256), 5)
    thin = [W.tiny(seed=s, n=n, bitwidth=3, n_streams=64, chunk_size=65536, table_log=12, p0=0.95).layers[0] for s, n in enumerate((12 * 65536 + 5, 9 * 65536))]
    return W.Workload("long", [thin[0], dense, thin[1]], 12, 64, 65536, "bf16")


@pytest.mark.parametrize("polls", [1, 2, 0])
def test_given_up_chunks_are_written_by_the_launch_behind(orc, polls):
    from helpers import oracle_encode
    w = _long_streams()
    c = oracle_encode(orc, w)
    fits = 32 * 138                                                # bits of a stream that LDS holds
    bits = (c.stream_hdr >> 16).reshape(-1, 64).max(axis=1) * 32
    assert (bits < fits).sum() > 20 and (bits > fits).sum() >= 1
    syms = [torch.from_numpy(x).to("cuda:0") for x in w.symbols()]
    f = torch.from_numpy(c.freqs.astype(np.uint32).view(np.int32)).to("cuda:0")
    one = orc.encode_layers([w.symbols()[0]], 12, 64, 65536)
    single = W.Workload("one", w.layers[:1], 12, 64, 65536, "bf16")
    try:
        B.lib().anszp_test_set_spin_limit(polls)
        _same(c, w, B.pack_layers_device(torch.cat(syms), [t.numel() for t in syms], f, 12, 64, 65536))
        _same(c, w, _pack_without_scratch(w, c))
        _same(one, single, B.pack_layer_device(syms[0], f[0], 12, 64, 65536))
        _same(one, single, _pack_layer_without_scratch(syms[0], f[0], 12, 64, 65536, len(one.payload) + 8))
    finally:
        B.lib().anszp_test_set_spin_limit(0)


@pytest.mark.parametrize("table_log,chunk", [(10, 1000), (12, 65536)])       # the last workgroup; the launch behind
def test_a_layer_of_bad_frequencies_in_front_of_given_up_chunks(orc, table_log, chunk):
    """Its chunks have no words but a place, which is not known in time either."""
    from helpers import oracle_encode
    layers = [W.tiny(seed=s, n=9 * chunk + 17 * s, bitwidth=4, n_streams=64, chunk_size=chunk, table_log=table_log, p0=0.9).layers[0] for s in range(5)]
    w = W.Workload("bad", layers, table_log, 64, chunk, "bf16")
    c = oracle_encode(orc, w)
    syms = w.symbols()
    s = torch.from_numpy(np.concatenate(syms)).to("cuda:0")
    for bad in ([1], [0, 1], [3, 4], [0, 4]):
        f = torch.from_numpy(c.freqs.astype(np.uint32).view(np.int32)).to("cuda:0").clone()
        f[bad, 0] += 1
        pack = lambda: B.pack_layers_device(s, [len(x) for x in syms], f, table_log, 64, chunk)
        expect = pack()
        assert expect[4].tolist() == [B.ST_BAD_FREQ, len(bad)] and 0 < int(expect[3].item()) < len(c.payload)
        try:
            B.lib().anszp_test_set_spin_limit(1)
            for _ in range(3):
                for a, b in zip(pack(), expect):
                    assert torch.equal(a, b)
        finally:
            B.lib().anszp_test_set_spin_limit(0)


def test_a_layer_packed_in_a_captured_graph(orc):
    """Scratch memory, counters and results belong to the graph: every replay packs the symbols that are there then."""
    sets = [W.tiny(seed=s, n=90001, bitwidth=4, n_streams=64, chunk_size=4096, table_log=11, p0=0.6).symbols()[0] for s in range(4)]
    freqs = B.normalize_freqs(np.bincount(np.concatenate(sets), minlength=256), 11)
    f = torch.from_numpy(freqs.astype(np.int32)).to("cuda:0")
    s = torch.from_numpy(sets[0]).to("cuda:0")
    expect = []
    for x in sets:
        expect.append([t.clone() for t in B.pack_layer_device(torch.from_numpy(x).to("cuda:0"), f, 11, 64, 4096)])
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        out = B.pack_layer_device(s, f, 11, 64, 4096)
    for k in (0, 1, 2, 3, 1, 0):
        s.copy_(torch.from_numpy(sets[k]).to("cuda:0"))
        g.replay()
        torch.cuda.synchronize()
        for a, b in zip(out, expect[k]):
            assert torch.equal(a, b), k
        B.pack_layer_device(s, f, 11, 64, 4096)                    # (eager work between the replays)
    assert tuple(expect[0][4].tolist()) == (0, 0)
