"""GPU parity of chunks that begin at any element of the output: layers of odd sizes one after the other, against the
oracle bit for bit.  The look-ahead kernel counts a chunk's positions from the multiple of 8 elements below its first
one; what can go wrong is the chunk's first eight elements, its end, and the neighbours' elements beside both."""
import numpy as np
import pytest
import torch

from paper_2406_06237_amd import binding as B
from paper_2406_06237_amd import workloads as W

from helpers import host_from_oracle, oracle_encode, oracle_expected

pytestmark = pytest.mark.gpu

# (first layer's size, the others' size, streams, chunk): every offset modulo 8 occurs; chunks of fewer than eight
# elements, of one slab (1024) and one more or less, of several slabs; more chunks than the chip has places (pairs)
CASES = [(1, 1027, 64, 4096), (3, 1024, 64, 1024), (7, 5, 64, 4096), (2049, 70001, 64, 65536), (5, 40003, 17, 16384),
         (9, 9001, 1, 16384), (13, 3000001, 64, 4099), (3, 2048 * 700 + 1, 33, 2051)]


@pytest.mark.parametrize("dtype", ["u8", "f32", "bf16"])
@pytest.mark.parametrize("table_log", [9, 12])
@pytest.mark.parametrize("first,size,n_streams,chunk", CASES)
def test_layers_at_odd_offsets(orc, dtype, table_log, first, size, n_streams, chunk):
    layers = [W.Layer(f"l{i}", (first if i == 0 else size,), 4, 8, 0.02 + 0.01 * i, W.peaked_geometric_pmf(16, 8, 0.7 if i % 2 else 0.3), 5 + i) for i in range(4)]
    _check(orc, W.Workload("offsets", layers, table_log, n_streams, chunk, dtype), dtype)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("channel", [1, 5, 8, 101])
def test_scales_per_channel_at_odd_offsets(orc, dtype, channel):
    rng = np.random.default_rng(channel)
    layers = [W.Layer(f"l{i}", (rows, channel), 4, 8, 0.0, W.laplace_pmf(16, 8, 1.0), 9 + i, channel_len=channel,
                      channel_scales=rng.uniform(0.005, 0.05, rows).astype(np.float32)) for i, rows in enumerate((3, 1001, 77, 503))]
    _check(orc, W.Workload("offsets", layers, 10, 64, 1000, dtype), dtype)


def _check(orc, w, dtype):
    c = oracle_encode(orc, w)
    _, expect = oracle_expected(orc, c, w, dtype)
    d = B.to_device(host_from_oracle(c, w))
    out = B.alloc_out(d, dtype)
    args = B.decode_args(d, out, dtype)
    plan = B.plan_decode(args, d.device)
    for how in ("automatic", "planned", "look-ahead"):
        out.view(torch.uint8).fill_(0xA5)
        if how == "planned":
            B.decode_planned_raw(args, plan, d.device)
        else:
            B.decode_raw(args, d.device, None if how == "automatic" else B.VARIANT_MERGED)
        assert d.read_status() == (0, 0), how
        got = B.bits_of(out)[:w.numel]
        bad = np.nonzero(got != expect)[0]
        assert len(bad) == 0, f"{how}: {len(bad)} mismatches, first at {bad[:5]}"
    # one chunk alone, between guard values: only its own elements are written
    guard = {"u8": 0xFF, "f32": 0xFFFFFFFF, "bf16": 0xFFFF}[dtype]
    for i in (0, 1, len(c.chunk_nsym) - 1):
        out.view(torch.uint8).fill_(0xFF)
        a = B.decode_args(d, out, dtype)
        a.chunks = d.chunks.data_ptr() + i * B.CHUNK_DTYPE.itemsize
        a.n_chunks = 1
        B.decode_raw(a, d.device, B.VARIANT_MERGED)
        assert d.read_status() == (0, 0)
        got = B.bits_of(out)[:w.numel]
        at, n = int(c.chunk_out_off[i]), int(c.chunk_nsym[i])
        assert np.array_equal(got[at:at + n], expect[at:at + n]), i
        assert bool((got[:at] == guard).all()) and bool((got[at + n:] == guard).all()), i
