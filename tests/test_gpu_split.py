"""GPU parity of the kernel that splits one stream over a workgroup, against the oracle bit for bit: streams around the
lengths at which the number of segments changes, tables from 2^5 to 2^12 states, more places than the pool of nodes holds
(long tables, segments much shorter than it takes two walks to meet), long runs that read no bits, buffers of symbols
that fill several times, chunks at odd offsets, scales per channel, and streams that do not end where they should."""
import numpy as np
import pytest
import torch

from paper_2406_06237_amd import binding as B
from paper_2406_06237_amd import workloads as W

from helpers import host_from_oracle, oracle_encode, oracle_expected

pytestmark = pytest.mark.gpu


def _decode(orc, layers, table_log, chunk, dtype, planned=False):
    w = W.Workload("split", layers, table_log, 1, chunk, dtype)
    c = oracle_encode(orc, w)
    _, expect = oracle_expected(orc, c, w, dtype)
    d = B.to_device(host_from_oracle(c, w))
    out = B.alloc_out(d, dtype)
    out.view(torch.uint8).fill_(0xA5)
    args = B.decode_args(d, out, dtype)
    if planned:
        B.decode_planned_raw(args, B.plan_decode(args, d.device), d.device)
    else:
        B.decode_raw(args, d.device)
    assert d.read_status() == (0, 0)
    bad = np.nonzero(B.bits_of(out)[:w.numel] != expect)[0]
    assert len(bad) == 0, f"{len(bad)} mismatches, first at {bad[:5]}"
    return c, d, expect


# symbols and bits of entropy such that the stream has about 0.5, 1, 1.5, 2, 4 and many times 2^table_log bits
@pytest.mark.parametrize("table_log", [5, 9, 10, 11, 12])
@pytest.mark.parametrize("n", [1300, 1700, 2200, 3300, 5200, 6900, 14000, 36864])
def test_lengths_and_tables(orc, table_log, n):
    for i, pmf in enumerate((W.laplace_pmf(16, 8, 0.9), W.peaked_geometric_pmf(256, 128, 0.55) if table_log > 8 else W.laplace_pmf(8, 4, 2.0))):
        _decode(orc, [W.Layer("one", (n,), 8, 8, 0.02, pmf, 3 + i)], table_log, 1 << 20, ("f32", "bf16")[i])


@pytest.mark.parametrize("dtype", ["u8", "f32", "bf16"])
@pytest.mark.parametrize("table_log,n,pmf", [
    (12, 300000, W.laplace_pmf(2, 1, 0.7)),                  # the longest stream that fits, many buffers of symbols
    (10, 350000, W.peaked_geometric_pmf(4, 2, 0.97)),        # runs that read no bits
    (12, 200000, W.peaked_geometric_pmf(16, 8, 0.99)),
    (9, 100001, W.laplace_pmf(64, 32, 4.0)),
    (12, 9000, np.ones(256) / 256), (10, 5000, np.ones(16) / 16),      # every symbol the same number of bits
])
def test_long_streams_and_odd_distributions(orc, dtype, table_log, n, pmf):
    _decode(orc, [W.Layer("one", (n,), 8, 8, 0.02, np.asarray(pmf), 11)], table_log, 1 << 20, dtype)


class _Exact(W.Layer):
    """Every symbol exactly as often as its share says, so that frequencies which are powers of two stay that."""
    def symbols(self):
        sym = np.repeat(np.arange(len(self.pmf)), (np.asarray(self.pmf) * self.numel).astype(int)).astype(np.uint8)
        assert len(sym) == self.numel
        return np.random.default_rng(self.seed).permutation(sym)


@pytest.mark.parametrize("table_log,pmf", [(r, q) for r in (5, 9, 12) for q in ([0.5, 0.5], [0.25] * 4, [1 / 16] * 16, [0.5, 0.25, 0.25],
                                                                             [0.25, 0.25] + [1 / 16] * 8, [1 / 256] * 256) if len(q) <= 1 << r])
def test_states_that_never_meet(orc, table_log, pmf):
    """A state keeps its upper bits: walks meet in the stream's own class of states and at its own bits, or not at all (and are
    started a second time there)."""
    for n, chunk in ((12288, 1 << 20), (5 * 12288, 12288)):
        _decode(orc, [_Exact("one", (n,), 8, 0, 0.02, np.asarray(pmf), 11)], table_log, chunk, "f32")


@pytest.mark.parametrize("planned", [False, True])
@pytest.mark.parametrize("dtype", ["u8", "f32", "bf16"])
def test_several_chunks_at_odd_offsets(orc, dtype, planned):
    layers = [W.Layer(f"l{i}", (n,), 4, 8, 0.02 + 0.01 * i, W.laplace_pmf(16, 8, 1.0 + 0.3 * i), 5 + i) for i, n in enumerate((5, 30011, 1, 20003, 40009))]
    _decode(orc, layers, 10, 16001, dtype, planned)


@pytest.mark.parametrize("channel", [1, 7, 342, 5000])
def test_scales_per_channel(orc, channel):
    rng = np.random.default_rng(channel)
    layers = [W.Layer(f"l{i}", (rows, channel), 4, 8, 0.0, W.laplace_pmf(16, 8, 1.0), 9 + i, channel_len=channel,
                      channel_scales=rng.uniform(0.005, 0.05, rows).astype(np.float32)) for i, rows in enumerate((3, 15000 // channel + 1, 21001 // channel + 1))]
    _decode(orc, layers, 10, 1 << 20, "bf16")
    _decode(orc, layers, 10, 1 << 20, "f32")


def test_streams_that_do_not_end_where_they_should(orc):
    """A flipped bit, another initial state, a length that is not the stream's: reported once per chunk, nothing written outside."""
    layers = [W.Layer("one", (n,), 4, 8, 0.02, W.laplace_pmf(16, 8, 1.0), 5) for n in (30000, 20001)]
    c, d, expect = _decode(orc, layers, 10, 1 << 20, "bf16")
    n0 = 30000
    payload, hdr = d.payload.clone(), d.stream_hdr.clone()
    cases = [("bit", d.payload, payload, 4 * 500, 0x10), ("state", d.stream_hdr, hdr, 0, 0x3), ("length", d.stream_hdr, hdr, 2, 0x1)]
    for name, t, keep, at, flip in cases:
        t[at] ^= flip
        buf = torch.full((d.host.numel + 128,), 0x5A5A, dtype=torch.int16, device="cuda:0")
        out = buf[64:64 + d.host.numel].view(torch.bfloat16)
        d.status.zero_()
        B.decode_raw(B.decode_args(d, out), d.device)
        st = d.read_status()
        assert st[1] == 1 and st[0] & (B.ST_BAD_STATE | B.ST_BAD_LENGTH | B.ST_BAD_DESC), (name, st)
        assert bool((buf[:64] == 0x5A5A).all()) and bool((buf[64 + d.host.numel:] == 0x5A5A).all()), name
        assert np.array_equal(B.bits_of(out)[n0:], expect[n0:]), name       # the other chunk is whole
        t.copy_(keep)
    # a chunk that says it has more or fewer symbols than its stream
    chunks = d.chunks.clone()
    for delta in (-3, 5):
        h = d.host.chunks.copy()
        h["n_symbols"][0] = n0 + delta
        d.chunks.copy_(torch.from_numpy(h.view(np.uint8).reshape(-1).copy()))
        d.status.zero_()
        out = B.alloc_out(d)
        B.decode_raw(B.decode_args(d, out), d.device)
        st = d.read_status()
        assert st[1] == 1 and st[0] & (B.ST_BAD_STATE | B.ST_BAD_LENGTH), (delta, st)
        d.chunks.copy_(chunks)


def test_random_words(orc):
    """Words that were never a stream: the walks go on through them, every loop ends, nothing is written outside."""
    c, d, _ = _decode(orc, [W.Layer("one", (30000,), 4, 8, 0.02, W.laplace_pmf(16, 8, 1.0), 5)], 10, 1 << 20, "bf16")
    g = torch.Generator(device="cuda:0").manual_seed(3)
    for _ in range(3):
        d.payload.copy_(torch.randint(0, 256, (d.payload.numel(),), dtype=torch.uint8, device="cuda:0", generator=g))
        buf = torch.full((d.host.numel + 128,), 0x5A5A, dtype=torch.int16, device="cuda:0")
        B.decode_raw(B.decode_args(d, buf[64:64 + d.host.numel].view(torch.bfloat16)), d.device)
        st = d.read_status()
        assert st[0] & (B.ST_BAD_STATE | B.ST_BAD_LENGTH), st
        assert bool((buf[:64] == 0x5A5A).all()) and bool((buf[64 + d.host.numel:] == 0x5A5A).all())
